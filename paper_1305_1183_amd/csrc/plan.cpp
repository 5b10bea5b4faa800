// plan.cpp -- data-dependency graph, fusion legality and plan enumeration.
//
// Section 4.2: the script's calls form a data-dependency graph; a *fusion* is
// a subgraph whose calls can share one kernel without changing the script's
// meaning; a plan (a "combination") covers every call with fusions and single
// calls. The legality rules follow Section 3.2:
//   R1  a kernel's call set is convex in the graph (no path leaves and
//       re-enters it), and the kernels of a plan form an acyclic graph;
//   R2  all calls of a kernel iterate over the same space -- calls of
//       different nesting depth (BLAS-1 vs BLAS-2) are never fused;
//   R3  a reduction result needs a global barrier, so it is not consumed in
//       the kernel that computes it (Section 3.2.2) -- except, as this
//       library's extension, as the additive y0 term of a reduction of the
//       same kind, which the last workgroup applies after its own barrier
//       (the "last running block" of Section 3.2.2);
//   R4  fusions that share no data save no transfers and are pruned.
#include <algorithm>
#include <functional>
#include <numeric>
#include <sstream>

#include "kf_internal.h"

namespace kf {

const char* op_name(Op op) {
    switch (op) {
        case Op::Scal: return "scal";
        case Op::Axpy: return "axpy";
        case Op::Dot: return "dot";
        case Op::Gemv: return "gemv";
        case Op::Gemtv: return "gemtv";
        case Op::Ger: return "ger";
    }
    return "?";
}

bool is_reduction(Op op) { return op == Op::Dot || op == Op::Gemv || op == Op::Gemtv; }

Space call_space(const Script& s, int c) {
    const Call& k = s.calls[c];
    Space sp;
    if (k.op == Op::Gemv || k.op == Op::Gemtv || k.op == Op::Ger) {
        const Value& A = s.values[k.in[0]];
        sp.mat = true;
        sp.a = A.rows;
        sp.b = A.cols;
    } else {
        sp.mat = false;
        sp.a = s.values[k.in[0]].n;
        sp.b = 0;
    }
    return sp;
}

// Data values (vectors, matrices) a call touches, inputs and output.
static std::vector<int> call_data(const Script& s, int ci) {
    std::vector<int> v;
    const Call& c = s.calls[ci];
    for (int i = 0; i < 3; ++i)
        if (c.in[i] >= 0) {
            VK k = s.values[c.in[i]].kind;
            if (k == VK::Vec || k == VK::Mat) v.push_back(c.in[i]);
        }
    VK k = s.values[c.out].kind;
    if (k == VK::Vec || k == VK::Mat) v.push_back(c.out);
    return v;
}

// Is the use of value `v` by call `d` the additive y0 term only?
static bool used_only_as_y0(const Call& d, int v) {
    if (d.alpha == v || d.beta == v) return false;
    if (d.in[0] == v || d.in[1] == v) return false;
    return d.in[2] == v;
}

std::string block_illegal_reason(const Script& s, const std::vector<int>& calls) {
    if (calls.empty()) return "empty";
    std::vector<char> in(s.calls.size(), 0);
    for (int c : calls) in[c] = 1;
    // R2: one iteration space.
    Space sp0 = call_space(s, calls[0]);
    for (int c : calls)
        if (!(call_space(s, c) == sp0)) return "R2: calls iterate over different spaces";
    // R3 (+ the same-kind y0 extension).
    for (int c : calls) {
        const Call& k = s.calls[c];
        if (!is_reduction(k.op)) continue;
        for (int d : s.values[k.out].consumers) {
            if (!in[d]) continue;
            const Call& kd = s.calls[d];
            bool ok = (k.op == Op::Gemv || k.op == Op::Gemtv) && kd.op == k.op &&
                      used_only_as_y0(kd, k.out);
            // R3'': a row dot may feed the row-indexed x of a gemtv when the kernel
            // keeps whole rows in one workgroup (row-resident schedule, cols <= 32768)
            if (!ok && k.op == Op::Gemv && kd.op == Op::Gemtv && kd.in[1] == k.out && kd.in[0] != k.out &&
                kd.in[2] != k.out && kd.alpha != k.out && kd.beta != k.out && call_space(s, c).b <= 32768 &&
                s.values[k.in[0]].dtype == KF_F32 && s.values[kd.in[0]].dtype == KF_F32)
                ok = true;
            if (!ok)
                return std::string("R3: result of ") + op_name(k.op) +
                       " consumed inside the kernel that reduces it";
        }
    }
    // R1: convexity -- no path from the set through an outside call back in.
    {
        std::vector<char> seen(s.calls.size(), 0);
        std::vector<int> stack;
        for (int c : calls)
            for (int d : s.values[s.calls[c].out].consumers)
                if (!in[d] && !seen[d]) { seen[d] = 1; stack.push_back(d); }
        while (!stack.empty()) {
            int d = stack.back();
            stack.pop_back();
            for (int e : s.values[s.calls[d].out].consumers) {
                if (in[e]) return "R1: a path leaves the kernel and re-enters it";
                if (!seen[e]) { seen[e] = 1; stack.push_back(e); }
            }
        }
    }
    // R4: connected through shared vectors or matrices.
    if (calls.size() > 1) {
        std::vector<int> comp(calls.size());
        std::iota(comp.begin(), comp.end(), 0);
        std::function<int(int)> find = [&](int x) { return comp[x] == x ? x : comp[x] = find(comp[x]); };
        for (size_t i = 0; i < calls.size(); ++i) {
            auto di = call_data(s, calls[i]);
            for (size_t j = i + 1; j < calls.size(); ++j) {
                auto dj = call_data(s, calls[j]);
                bool share = false;
                for (int a : di)
                    for (int b : dj)
                        if (a == b) share = true;
                if (share) comp[find((int)i)] = find((int)j);
            }
        }
        int root = find(0);
        for (size_t i = 1; i < calls.size(); ++i)
            if (find((int)i) != root) return "R4: the calls share no vector or matrix";
    }
    return "";
}

bool partition_acyclic(const Script& s, const std::vector<int>& part, int nk) {
    std::vector<std::set<int>> succ(nk);
    for (size_t c = 0; c < s.calls.size(); ++c)
        for (int d : s.values[s.calls[c].out].consumers)
            if (part[d] != part[c]) succ[part[c]].insert(part[d]);
    std::vector<int> indeg(nk, 0);
    for (int k = 0; k < nk; ++k)
        for (int t : succ[k]) indeg[t]++;
    std::vector<int> q;
    for (int k = 0; k < nk; ++k)
        if (!indeg[k]) q.push_back(k);
    int seen = 0;
    while (!q.empty()) {
        int k = q.back();
        q.pop_back();
        ++seen;
        for (int t : succ[k])
            if (--indeg[t] == 0) q.push_back(t);
    }
    return seen == nk;
}

static std::vector<int> canonical(const std::vector<int>& part) {
    std::map<int, int> ren;
    std::vector<int> out(part.size());
    for (size_t i = 0; i < part.size(); ++i) {
        auto it = ren.find(part[i]);
        if (it == ren.end()) it = ren.emplace(part[i], (int)ren.size()).first;
        out[i] = it->second;
    }
    return out;
}

std::vector<std::vector<int>> enumerate_partitions(const Script& s, int max_plans) {
    const int n = (int)s.calls.size();
    std::vector<std::vector<int>> result;
    if (n == 0) return result;
    // Candidate blocks: legal subsets of each iteration-space group.
    std::map<Space, std::vector<int>> groups;
    for (int c = 0; c < n; ++c) groups[call_space(s, c)].push_back(c);
    std::vector<std::vector<std::vector<int>>> blocks_with(n);  // blocks whose min call is c
    for (auto& g : groups) {
        const auto& mem = g.second;
        const int gsz = (int)mem.size();
        if (gsz > 20) {
            // Too many subsets to list: only singletons.
            for (int c : mem) blocks_with[c].push_back({c});
            continue;
        }
        for (uint32_t mask = 1; mask < (1u << gsz); ++mask) {
            std::vector<int> b;
            for (int i = 0; i < gsz; ++i)
                if (mask & (1u << i)) b.push_back(mem[i]);
            if (b.size() == 1 || block_illegal_reason(s, b).empty()) blocks_with[b[0]].push_back(b);
        }
    }
    // Exact covers by blocks, then the acyclicity check of the plan.
    const size_t hard_cap = 200000;
    std::vector<int> part(n, -1);
    int nk = 0;
    std::function<void(int)> rec = [&](int first) {
        if (result.size() >= hard_cap) return;
        while (first < n && part[first] >= 0) ++first;
        if (first == n) {
            if (partition_acyclic(s, part, nk)) result.push_back(canonical(part));
            return;
        }
        for (const auto& b : blocks_with[first]) {
            bool free_ = true;
            for (int c : b)
                if (part[c] >= 0) { free_ = false; break; }
            if (!free_) continue;
            for (int c : b) part[c] = nk;
            ++nk;
            rec(first + 1);
            --nk;
            for (int c : b) part[c] = -1;
        }
    };
    rec(0);
    auto nkern = [](const std::vector<int>& p) { return *std::max_element(p.begin(), p.end()) + 1; };
    std::stable_sort(result.begin(), result.end(), [&](const std::vector<int>& a, const std::vector<int>& b) {
        int ka = nkern(a), kb = nkern(b);
        if (ka != kb) return ka < kb;
        return a < b;
    });
    if (max_plans > 0 && (int)result.size() > max_plans) result.resize(max_plans);
    return result;
}

std::vector<int> fused_partition(const Script& s) {
    auto all = enumerate_partitions(s, 1);
    if (all.empty()) return unfused_partition(s);
    return all[0];
}

std::vector<int> unfused_partition(const Script& s) {
    std::vector<int> p(s.calls.size());
    std::iota(p.begin(), p.end(), 0);
    return p;
}

std::vector<std::vector<int>> kernels_in_order(const Script& s, const std::vector<int>& part) {
    int nk = part.empty() ? 0 : *std::max_element(part.begin(), part.end()) + 1;
    std::vector<std::vector<int>> members(nk);
    for (size_t c = 0; c < part.size(); ++c) members[part[c]].push_back((int)c);
    std::vector<std::set<int>> succ(nk);
    std::vector<int> indeg(nk, 0);
    for (size_t c = 0; c < s.calls.size(); ++c)
        for (int d : s.values[s.calls[c].out].consumers)
            if (part[d] != part[c] && succ[part[c]].insert(part[d]).second) indeg[part[d]]++;
    std::vector<std::vector<int>> order;
    std::set<std::pair<int, int>> ready;  // (first call, kernel)
    for (int k = 0; k < nk; ++k)
        if (!indeg[k]) ready.insert({members[k][0], k});
    while (!ready.empty()) {
        int k = ready.begin()->second;
        ready.erase(ready.begin());
        order.push_back(members[k]);
        for (int t : succ[k])
            if (--indeg[t] == 0) ready.insert({members[t][0], t});
    }
    return order;
}

int dtype_size(int dtype) { return dtype == KF_BF16 ? 2 : dtype == KF_FP8_E4M3 ? 1 : 4; }

int kernel_unit_elems(const Script& s, const std::vector<int>& calls, int req) {
    int es = 4;
    bool ger_q = false;
    for (int c : calls) {
        const Value& A = s.values[s.calls[c].in[0]];
        if (A.kind == VK::Mat) es = std::min(es, dtype_size(A.dtype));
        if (A.kind == VK::Mat && A.dtype != KF_F32 && s.calls[c].op == Op::Ger) ger_q = true;
    }
    // req: 4 = narrow units (four elements per lane and load), 16 = one
    // 16-byte load per lane; 0 = automatic. Automatically, a kernel that
    // expands a quantised matrix into an FP32 one (ger) takes narrow units so
    // that its FP32 stores stay 16 bytes per lane and contiguous across the
    // wave; other kernels take 16-byte loads.
    if (es == 4 || req == 4) return 4;
    if (req == 16) return 16 / es;
    if (ger_q) return 4;
    return 16 / es;
}

bool kernel_has_quantized(const Script& s, const std::vector<int>& calls) {
    for (int c : calls) {
        const Value& A = s.values[s.calls[c].in[0]];
        if (A.kind == VK::Mat && A.dtype != KF_F32) return true;
    }
    return false;
}

MatParams default_mat_params(int64_t rows, int64_t cols, const MatParams& req, int e_per_unit) {
    MatParams p = req;
    if (p.k <= 0) p.k = 1;
    if (p.waves <= 0) p.waves = 4;
    if (p.group <= 0) p.group = 4;
    const int unit = p.waves * p.group;
    if (p.rows <= 0) {
        const int64_t C = 64LL * e_per_unit * p.k;
        const int64_t S = (cols + C - 1) / C;
        // Aim for about 2048 workgroups (8 per CU) with at most 512 rows each.
        int64_t want_nb = (2048 + S - 1) / S;
        int64_t r = (rows + want_nb - 1) / want_nb;
        r = ((r + unit - 1) / unit) * unit;
        if (r < unit) r = unit;
        if (r > 512) r = (512 / unit) * unit;
        if (r < unit) r = unit;
        p.rows = (int)r;
    }
    return p;
}

// The library's own strip geometry for a kernel whose caller asks for none: k, W
// and G, and a number of row blocks that gives every CU the stated waves. Each
// line was timed over square and uneven shapes from 128 to 32768 against ten to
// fourteen others (whole plans, three inputs in turn; us at the sizes named):
//  - small matrices (6M elements, about what stays in L2) are bound by latency and
//    by the finishing launch, which wants few row blocks: four rows per step and
//    wave. BiCGK n = 1024 5.7 (sixteen waves, two float4: 7.2); 2048 8.9 (10.4).
//  - kernels that store a matrix mix reads and writes, and DRAM serves that best
//    from eight waves a CU: GEMVER's first kernel n = 16384 346 (sixteen waves of
//    the next line 413, 2048 small workgroups 361). Rows that do not start on
//    1 KiB boundaries take two float4 per lane, as strip edges then cost part of a
//    line on each side: n = 9000 131 (one float4: 163). Rows of fewer than 256 columns
//    fill part of a strip and want sixteen waves a CU: 89702 x 100 32 (eight: 44); so do
//    BF16 and FP8 sources, which read less than they store, up to 400M elements: BF16 n =
//    4000 28 (32), 6000 x 30000 247 (273), 24000 x 20100 803 (646). Without column sums
//    there are no partials to save, and narrow matrices keep the small workgroups: ger
//    89702 x 100 23 (40), 20000 x 700 29 (31), 9000 163 (128); BF16 and FP8 up to 40M
//    elements: BF16 2000 x 8000 21 (27), 6000 53 (56), 9000 133 (124).
//  - other FP32 kernels: one workgroup of sixteen waves per CU, 2 KiB strips. BiCGK
//    n = 16384 165 (2048 workgroups of four waves: 186), 5003 21.3 (26.5), 12001 94
//    (124), 700 x 16000 12.5 (22.6).
//  - BF16 and FP8 in 16-byte units: 24 and 20 waves per CU, as many as their registers
//    allow, hide the conversion. BiCGK n = 16384 FP8 54 (79), BF16 90 (96). One or two
//    strips leave row blocks only; sixteen waves a workgroup then keep their number down
//    (FP8 50000 x 500 21, 50). In requested units of four elements, which carry a quarter
//    or half of the bytes, 24 waves of two rows from 40M elements on: FP8 n = 16384 60 (the
//    line before 95, small workgroups 77), n = 8192 22 (30, 24), 5003 18.4 (16.9, 20).
// The number of workgroups stays within one round of the chip: a few more would run in
// a second, nearly empty one (BiCGK n = 10007 98 with 260 workgroups, 66 with 240; n =
// 24000 493 with 282, 354 with 235).
//
// A wave adds its rows of a column in plain FP32 before (sum, error) pairs take over:
// no longer chains of them than in the small workgroups (default_mat_params, `chain`
// rows), so that larger blocks do not cost precision. Past that, in this order:
//  - steps of two or four rows enter pairs one by one, where the registers are there
//    (GEMVER n = 16384 509 us, 511 in plain FP32);
//  - a step's rows are summed first, which halves the chain (BiCGK 20000 x 700 17.7 us,
//    18.0 with one row a step): 1.5 + n / 4 squared roundings a row over n rows instead
//    of (n + 1) / 2;
//  - a workgroup takes its rows in several blocks, one after another, each with its own
//    partials, and no more of them than the small workgroups have (BiCGK n = 32768 666
//    us, 688 with pairs every 128 rows; FP8 178 and 258). So do blocks of more than 4096
//    rows, whose vectors are staged in LDS (GEMVER n = 24000 1230 us; 1500 with 282
//    workgroups of one block each).
static MatParams library_mat_params(int64_t rows, int64_t cols, int E, bool stores, bool column_sums, bool quantized) {
    MatParams p;
    const int64_t few = default_mat_params(rows, cols, MatParams(), E).rows, chain = few / 4;
    const int64_t by_row = chain + chain / 16, by_step = (11 * chain - 17) / 5;   // rows of a wave, within 5% of its error
    int per_cu;
    const double elems = (double)rows * (double)cols;
    const bool small = elems <= 6e6, general = !small && !stores, ragged = quantized && cols % 256 != 0;
    if (small) { p.k = 1; p.waves = 8; p.group = 4; per_cu = 16; }
    else if (stores && !column_sums && (cols < 1024 || (ragged && elems <= 4e7)))
        return default_mat_params(rows, cols, p, E);
    else if (stores && (cols < 256 || (ragged && column_sums && elems <= 4e8))) { p.k = 1; p.waves = 8; p.group = 4; per_cu = 16; }
    else if (stores) { const bool line = cols % 256 == 0; p.k = line ? 1 : 2; p.waves = 8; p.group = line ? 4 : 2; per_cu = 8; }
    else if (E == 4 && quantized && elems > 4e7) { p.k = 2; p.waves = 8; p.group = 2; per_cu = 24; }
    else if (E == 4) { p.k = 2; p.waves = 16; p.group = 1; per_cu = 16; }
    else if (cols <= 2 * 64 * E) { p.k = 1; p.waves = 16; p.group = 2; per_cu = 16; }
    else { p.k = 1; p.waves = 4; p.group = 2; per_cu = E == 16 ? 20 : 24; }
    const int64_t C = 64LL * E * p.k, S = (cols + C - 1) / C, nb = std::max<int64_t>(1, 256 * per_cu / (S * p.waves));
    auto block_rows = [&](int64_t n) {   // rows of each of n blocks, whole steps
        const int64_t r = (rows + n - 1) / n, unit = p.waves * p.group;
        return std::max<int64_t>((r + unit - 1) / unit * unit, p.waves * std::max(4, p.group));
    };
    int64_t r = block_rows(nb);
    auto wave_rows = [&]() { return (r + p.waves - 1) / p.waves; };
    if (column_sums && general && E == 4 && wave_rows() > by_row && wave_rows() <= by_step) {
        p.group = 2;
        r = block_rows(nb);
    }
    int64_t most = 4096;
    if (!column_sums) {
    } else if (general && p.group > 1) {
        p.sums = ColSum::Steps;
        most = std::min(most, by_step * p.waves);
    } else if (p.group == 1) {
        most = std::min(most, by_row * p.waves);
    } else if (wave_rows() > chain) {
        // a lane of sixteen FP8 columns has no registers for pairs beside the stored matrix
        // (GEMVER's first kernel at n = 16384 1314 us, small workgroups 995)
        if (stores && E == 16) return default_mat_params(rows, cols, MatParams(), E);
        p.sums = ColSum::Pairs;
    }
    if (r > most) {
        p.turns = (int)((r + most - 1) / most);
        p.blocks = std::min(nb * p.turns, (rows + few - 1) / few);
        r = block_rows(p.blocks);
    }
    p.rows = (int)r;
    p.sub = p.k;
    return p;
}

bool library_geometry(const MatParams& p) { return p.sched == 0 && p.k <= 0 && p.waves <= 0 && p.group <= 0 && p.rows <= 0; }

MatParams kernel_mat_params(const Script& s, const std::vector<int>& calls, const MatParams& req) {
    const Space sp = call_space(s, calls[0]);
    const int E = kernel_unit_elems(s, calls, req.unit);
    // A plan compiled for shapes up to the declared one keeps the small workgroups: the
    // blocks that fill the chip at the declared shape are few at a smaller one (BiCGK
    // declared 16384 x 16384, run at 4096 x 4096 29 us, with its geometry 92; at 16384 176, 174).
    if (req.dyn) return default_mat_params(sp.a, sp.b, req, E);
    const std::set<int> mine(calls.begin(), calls.end());
    std::set<int> mats, cols, rows;
    int gemtv = 0;
    bool stores = false, ger = false;
    for (int c : calls) {
        const Call& k = s.calls[c];
        const int prod = s.values[k.in[0]].producer;
        if (prod < 0 || !mine.count(prod)) {
            mats.insert(k.in[0]);
            if (s.values[k.in[0]].scale >= 0) rows.insert(s.values[k.in[0]].scale);
        }
        if (k.op == Op::Gemtv) { ++gemtv; rows.insert(k.in[1]); }
        if (k.op == Op::Gemv) cols.insert(k.in[1]);
        if (k.op != Op::Ger) continue;
        ger = true;
        rows.insert(k.in[1]);
        cols.insert(k.in[2]);
        const Value& o = s.values[k.out];
        stores = stores || o.output;
        for (int d : o.consumers) stores = stores || !mine.count(d);
    }
    MatParams p = library_mat_params(sp.a, sp.b, E, stores, gemtv > 0, kernel_has_quantized(s, calls));
    // kernels of so many operands that a lane's rows, vectors and accumulators
    // outgrow the registers (128 with sixteen waves in a workgroup, 256 with
    // eight) or the staged vectors and wave sums the LDS keep the small workgroups
    const int K = p.k * E / 4, sets = p.sums == ColSum::Pairs ? 3 : 1;
    const int regs = 4 * K * (p.group * (int)mats.size() + (int)cols.size() + gemtv * sets + (ger ? 1 : 0));
    const int64_t lds = (int64_t)rows.size() * p.rows * 4 + (int64_t)gemtv * p.waves * std::min(sets, 2) * 64 * K * 16;
    // (kernels that store a matrix have one workgroup on a CU, the others two)
    if (regs > (p.waves > 8 ? 72 : 168) || lds > (stores ? 112 : 72) * 1024) p = default_mat_params(sp.a, sp.b, MatParams(), E);
    p.unit = req.unit;
    if (library_geometry(req)) return p;
    // a requested point that is the library's own gives the library's kernel
    MatParams q = default_mat_params(sp.a, sp.b, req, E);
    if (q.k == p.k && q.waves == p.waves && q.group == p.group && q.rows == p.rows) {
        q.sums = p.sums;
        q.turns = p.turns;
        q.sub = p.sub;
        q.blocks = p.blocks;
    }
    return q;
}

VecParams default_vec_params(int64_t n, const VecParams& req) {
    VecParams p = req;
    if (p.unroll <= 0) p.unroll = 4;
    if (p.threads <= 0) p.threads = 256;
    int64_t n4 = n / 4;
    int64_t need = (n4 + (int64_t)p.threads * p.unroll - 1) / ((int64_t)p.threads * p.unroll);
    if (need < 1) need = 1;
    if (p.grid <= 0) p.grid = 2048;
    if (need < p.grid) p.grid = (int)need;
    return p;
}

}  // namespace kf
