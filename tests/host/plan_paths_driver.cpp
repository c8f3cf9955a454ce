// Checks of the plan code's choices on a recording HIP runtime (fake_hip.hpp):
// one check per name, picked by the first argument.  Exit status 0 if it holds.
#include "fake_hip.hpp"

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <tuple>

#include "nr_internal.hpp"
#include "nufft_resample.h"

namespace {

struct Bank {
    std::vector<nr_segment> segs;
    std::vector<nr_template> tmpls;
};

// n_seg segments of L samples at fs; n_mc chirp masses x n_sub sub-bands of K bins of df from 40 Hz on
Bank bank(int n_seg, int64_t L, double fs, int n_mc, int n_sub, int K, double df, double mc0 = 1e-3, double mc1 = 1e-1)
{
    Bank b;
    for (int i = 0; i < n_seg; ++i) b.segs.push_back({i * L, L, fs, (double)(i * L) / fs});
    for (int m = 0; m < n_mc; ++m)
        for (int s = 0; s < n_sub; ++s) {
            nr_template t{};
            t.mc_msun = mc0 * std::pow(mc1 / mc0, n_mc > 1 ? m / (n_mc - 1.0) : 0.0);
            t.f_lo = 40.0 + s;
            t.f0 = t.f_lo + 0.5 * K * df;
            t.df = df;
            t.n_bins = K;
            b.tmpls.push_back(t);
        }
    return b;
}

nr_status plan(nr_plan* p, const Bank& b, double tol, const nr_options& o)
{
    return nufft_resample_plan(p, b.segs.data(), (int)b.segs.size(), b.tmpls.data(), (int)b.tmpls.size(), nullptr, 0,
                               tol, &o);
}

nr_options options(int precision)
{
    nr_options o;
    nufft_resample_default_options(&o);
    o.precision = precision;
    return o;
}

bool has_nodes(nr_plan p)
{
    nr_plan_info info;
    nufft_resample_query(p, &info);
    for (int c = 0; c < info.n_classes; ++c) {
        nr_node_info n;
        nufft_resample_query_nodes(p, c, &n);
        if (n.width) return true;
    }
    return false;
}

// A strict plan accepts the tolerances that it accepts on the samples: the node
// path's tau series spans more than the segment and may be longer.
int strict()
{
    int refused = 0, with_nodes = 0, accepted = 0;
    for (double mc1 : {2e-2, 5e-2, 1e-1})
        for (double tol = 1e-11; tol < 2e-10; tol *= 1.02) {
            const Bank b = bank(2, 7680, 256.0, 24, 2, 30, 1.0 / 30, 1e-2, mc1);
            nr_options o = options(NR_FP64);
            o.strict = 1;
            nr_plan p = nullptr, q = nullptr;
            const nr_status a = plan(&p, b, tol, o);
            o.method = NR_METHOD_CELLRUN;
            const nr_status s = plan(&q, b, tol, o);
            if (a != s) {
                std::printf("mc %g tol %g: status %d, %d on samples (%s)\n", mc1, tol, (int)a, (int)s,
                            nufft_resample_last_error(nullptr));
                ++refused;
            }
            if (s == NR_OK) ++accepted;
            if (a == NR_OK && has_nodes(p)) ++with_nodes;
            nufft_resample_destroy(p);
            nufft_resample_destroy(q);
        }
    std::printf("%d accepted on samples, %d with nodes, %d differ\n", accepted, with_nodes, refused);
    return refused || !accepted || !with_nodes;
}

// Whichever allocation of the node path fails, the plan is built on the samples
// and its calls do not meet the allocation's error again.
int fallback()
{
    const Bank b = bank(2, 7680, 256.0, 24, 2, 30, 1.0 / 30);
    const nr_options o = options(NR_FP32);
    nr_plan p = nullptr;
    int64_t before = fake_hip::allocations;
    if (plan(&p, b, 1e-6, o) != NR_OK || !has_nodes(p)) return 1;
    const int64_t n = fake_hip::allocations - before;
    nufft_resample_destroy(p);
    std::vector<float> strain(2 * 7680), stat(48 * 30), power(48 * 2 * 30);
    int bad = 0, samples = 0;
    for (int64_t k = 0; k < n; ++k) {
        fake_hip::fail_at = fake_hip::allocations + k;
        const nr_status st = plan(&p, b, 1e-6, o);
        fake_hip::fail_at = -1;
        const nr_status e = st != NR_OK ? st : nufft_resample_execute(p, strain.data(), nullptr, power.data(), nullptr);
        const nr_status u =
            st != NR_OK ? st : nufft_resample_semicoherent_sum(p, strain.data(), nullptr, stat.data(), nullptr);
        if (st != NR_OK || e != NR_OK || u != NR_OK) {
            std::printf("allocation %d: plan %d, execute %d, sum %d: %s\n", (int)k, (int)st, (int)e, (int)u,
                        st != NR_OK ? nufft_resample_last_error(nullptr) : nufft_resample_last_error(p));
            ++bad;
        } else if (!has_nodes(p)) {
            ++samples;
        }
        nufft_resample_destroy(p);
        (void)hipGetLastError();
    }
    std::printf("%d allocations, %d fall back, %d bad\n", (int)n, samples, bad);
    return bad || samples != n;
}

// A large grid whose strips would fill the LDS to the last byte leaves the
// kernel's 16 static bytes no room: the plan takes the samples.  Bins ever
// further apart pass that size (n = 240 and four strips of 5060 cells).
int full_lds()
{
    int met = 0, over = 0, below = 0;
    std::vector<float> strain(491520), power(64 * 120);
    for (double df = 2.80; df < 2.8060 && !over; df += 2e-5) {
        Bank b = bank(1, 491520, 16384.0, 64, 1, 120, df);
        for (nr_template& t : b.tmpls) t.mc_msun = 0.0;
        nr_plan p = nullptr;
        if (plan(&p, b, 1e-6, options(NR_FP32)) != NR_OK) return 1;
        fake_hip::launches.clear();
        if (nufft_resample_execute(p, strain.data(), nullptr, power.data(), nullptr) != NR_OK) return 1;
        bool fft = false;
        for (const fake_hip::Launch& l : fake_hip::launches)
            if (l.is("node_spread_fft")) {
                fft = true;
                over += l.lds + 16 > 160 * 1024;
                below += l.lds > 160 * 1024 - 256;
                std::printf("df %.5f lds %zu\n", df, l.lds);
            }
        met += !fft;
        nufft_resample_destroy(p);
    }
    std::printf("%d plans just below, %d on samples, %d over\n", below, met, over);
    return over || !below || !met;
}

// The launches of more node instances, or filter work, than one launch's 2^32
// threads hold are split, each piece with its own records.
int large_launches()
{
    fake_hip::arg_bytes = sizeof(nr::NodeArgs);
    nr::NodeArgs a{};
    a.inst = reinterpret_cast<const nr::InstDev*>(uintptr_t(1) << 40);   // (never read here)
    a.count = (int64_t(1) << 24) + 5;
    a.n = 144;
    a.w = 8;
    a.strip = 40;
    int bad = 0;
    for (const int small : {0, 1}) {
        a.mtiles = small ? 4 : 0;
        a.count = (small ? int64_t(1) << 28 : int64_t(1) << 24) + 5;
        fake_hip::launches.clear();
        bad += nr::launch_node_spread(a, 0, nr::EpilogueOut{}, nullptr) != hipSuccess;
        int64_t at = 0;
        for (const fake_hip::Launch& l : fake_hip::launches) {
            nr::NodeArgs q;
            std::memcpy(&q, l.arg.data(), sizeof q);
            bad += q.inst != a.inst + at || (int64_t)l.grid.x * (small ? nr::kNodeBatch : 1) < q.count;
            at += q.count;
        }
        bad += at != a.count;
    }
    nr::FilterLaunch f{};
    f.items = reinterpret_cast<const nr::FilterItem*>(uintptr_t(1) << 40);
    f.count = (int64_t(1) << 24) + 5;
    f.tiles = 1;
    f.images = 5;
    f.lds = 60000;
    fake_hip::launches.clear();
    fake_hip::arg_bytes = sizeof(f.items);
    bad += nr::launch_node_filter(f, nullptr, nullptr, 0, 0, nullptr) != hipSuccess;
    int64_t at = 0;
    for (const fake_hip::Launch& l : fake_hip::launches) {
        const nr::FilterItem* items;
        std::memcpy(&items, l.arg.data(), sizeof items);
        bad += items != f.items + at;
        at += l.grid.x;
    }
    bad += at != f.count;
    std::printf("%d bad\n", bad);
    return bad;
}

// What the tuner times is what the tuned plan runs: with cell runs made the
// cheapest, the plan's spread launch (grid, LDS, waves an instance, records) is
// among those of the mini-plans.
int tuner()
{
    fake_hip::arg_bytes = sizeof(nr::SpreadArgs);
    fake_hip::cost = [](const fake_hip::Launch& l) {
        return l.is("spread_runs") ? 0.1 : l.is("spread") || l.is("tau") ? 10.0 : 0.1;
    };
    int bad = 0;
    // (a shape's choice is kept for the process: a length of its own for each)
    int64_t L = 7680;
    for (const int precision : {NR_FP32, NR_FP64, NR_AUTO})
        for (const int n : {1, 16, 300}) {
            L += 4;
            Bank b = bank(n, L, 256.0, 1, 1, 600, 1.0 / 30);
            nr_options o = options(precision);
            o.tune = 1;
            fake_hip::launches.clear();
            nr_plan p = nullptr;
            if (plan(&p, b, precision == NR_FP64 ? 1e-9 : 1e-6, o) != NR_OK) return 1;
            const std::vector<fake_hip::Launch> timed = fake_hip::launches;
            std::vector<double> strain(n * L), power(n * 600);
            fake_hip::launches.clear();
            if (nufft_resample_execute(p, strain.data(), nullptr, power.data(), nullptr) != NR_OK) return 1;
            int runs = 0;
            for (const fake_hip::Launch& l : fake_hip::launches)
                if (l.is("spread_runs")) {
                    const auto shape = [](const fake_hip::Launch& q) {
                        nr::SpreadArgs a;
                        std::memcpy(&a, q.arg.data(), sizeof a);
                        return std::make_tuple(q.kernel, q.grid.x, q.lds, a.count, a.n, a.parts, a.rec_stride, a.rec_shift);
                    };
                    bool found = false;
                    for (const fake_hip::Launch& q : timed) found = found || (q.is("spread_runs") && shape(q) == shape(l));
                    bad += !found;
                    ++runs;
                }
            std::printf("precision %d, %d instances: %d cell-run launches, %d bad so far\n", precision, n, runs, bad);
            if (!runs) return 1;
            nufft_resample_destroy(p);
        }
    return bad;
}

// A merged launch takes a class below the occupancy that its own LDS allows only
// if every workgroup of the launch is resident at once.
int groups()
{
    fake_hip::arg_bytes = sizeof(nr::SpreadTable);
    const auto tier = [](size_t lds) { return (int64_t)std::min<size_t>(8, 160 * 1024 / std::max<size_t>(lds, 1)); };
    int bad = 0, merged = 0, lowered = 0;
    // templates of 30 bins (2 KB of LDS), of 1200 (77 KB) and of 1250 (80 KB) in every order
    const int K[3] = {30, 1200, 1250};
    const int orders[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};
    for (const auto& order : orders)
        for (int many = 0; many < 4; ++many) {           // which of them has 4096 (3: none)
            Bank b = bank(1, 7680, 256.0, 1, 1, 30, 1.0 / 30);
            const nr_template t = b.tmpls[0];
            b.tmpls.clear();
            for (const int k : order)
                for (int q = 0; q < (k == many ? 4096 : 8); ++q) {
                    b.tmpls.push_back(t);
                    b.tmpls.back().n_bins = K[k];
                }
            nr_options o = options(NR_FP32);
            o.method = NR_METHOD_FUSED;
            o.parts = 1;
            nr_plan p = nullptr;
            if (plan(&p, b, 1e-6, o) != NR_OK) return 1;
            std::vector<float> strain(7680);
            float power = 0.0f;                          // (launches write nothing here)
            fake_hip::launches.clear();
            if (nufft_resample_execute(p, strain.data(), nullptr, &power, nullptr) != NR_OK) return 1;
            for (const fake_hip::Launch& l : fake_hip::launches) {
                if (!l.is("spread") || !l.is("SpreadTable")) continue;
                nr::SpreadTable tab;
                std::memcpy(&tab, l.arg.data(), sizeof tab);
                ++merged;
                for (int c = 0; c < tab.ncls; ++c) {
                    const nr::SpreadArgs& a = tab.a[c];
                    const size_t own = nr::spread_lds_bytes(0, a.n, a.epi_fused && a.parts == 1);
                    if (tier(own) <= tier(l.lds)) continue;
                    ++lowered;
                    if (l.grid.x > 256 * tier(l.lds)) {
                        std::printf("order %d %d %d, many %d: %u workgroups of %zu bytes hold a class of %zu\n", order[0],
                                    order[1], order[2], many, l.grid.x, l.lds, own);
                        ++bad;
                    }
                }
            }
            nufft_resample_destroy(p);
        }
    std::printf("%d merged launches, %d classes below their occupancy, %d wrongly\n", merged, lowered, bad);
    return bad || !merged || !lowered;
}

// Workgroups a segment of the lane-major strain copies: few entries a thread where
// compute units would idle or the strain passes the last-level cache, else more.
int copies()
{
    const struct {
        int n;
        int64_t L;
        double fs;
        int precision;
        unsigned y;
    } want[] = {{1, 7680, 256.0, NR_FP32, 8},       {128, 7680, 256.0, NR_FP32, 8},    {512, 7680, 256.0, NR_FP32, 2},
                {2048, 7680, 256.0, NR_FP32, 2},    {4096, 7680, 256.0, NR_AUTO, 8},   {2048, 1920, 64.0, NR_FP64, 1},
                {128, 30720, 1024.0, NR_FP32, 8},   {512, 30720, 1024.0, NR_FP32, 30}};
    int bad = 0;
    for (const auto& c : want) {
        Bank b = bank(c.n, c.L, c.fs, 1, 1, 30, 1.0 / 30);
        nr_options o = options(c.precision);
        o.method = NR_METHOD_FUSED;
        o.parts = 1;
        nr_plan p = nullptr;
        if (plan(&p, b, c.precision == NR_FP64 ? 1e-9 : 1e-6, o) != NR_OK) return 1;
        std::vector<double> strain(1);
        float power = 0.0f;
        fake_hip::launches.clear();
        if (nufft_resample_execute(p, strain.data(), nullptr, &power, nullptr) != NR_OK) return 1;
        for (const fake_hip::Launch& l : fake_hip::launches)
            if (l.is("strain_lane_major") && (l.grid.x != (unsigned)c.n || l.grid.y != c.y)) {
                std::printf("%d segments of %d: %u x %u\n", c.n, (int)c.L, l.grid.x, l.grid.y);
                ++bad;
            }
        nufft_resample_destroy(p);
    }
    return bad;
}

// Which of the shapes that the GPU tests of records plan take them: all but the
// segment of three samples, whose cells hold fewer than 1.5 each.
int records()
{
    fake_hip::arg_bytes = sizeof(nr::SpreadArgs);
    const struct {
        int n;
        int64_t L;
        double fs;
        int K;
        double df;      // <= 0: 1 / T
        bool rec;
    } shapes[] = {{1, 3, 256.0, 1, 0.0, false},      {3, 65, 256.0, 16, 0.0, true},
                  {2, 7681, 256.0, 600, 0.0, true},  {5, 2560, 256.0, 200, 0.0, true},
                  {4, 7679, 256.0, 32, 8 / 30., true}, {2, 30719, 1024.0, 40, 0.0, true},
                  {130, 4099, 128.0, 130, 1 / 16., true}, {700, 1025, 128.0, 140, 1 / 8., true},
                  {1, 3, 256.0, 2, 1e-3, false},     {1, 4, 256.0, 2, 1e-3, true},
                  {1, 5, 256.0, 2, 1e-3, true},      {1, 7, 256.0, 2, 1e-3, true},
                  {1, 63, 256.0, 2, 1e-3, true},     {1, 64, 256.0, 2, 1e-3, true}};
    int bad = 0;
    for (const auto& q : shapes)
        for (const double tol : {1e-3, 1e-6, 1e-9, 1e-12}) {
            Bank b = bank(2, q.L, q.fs, q.n, 1, q.K, q.df, 1e-4, 1e-3);
            for (nr_template& t : b.tmpls) t.f0 = t.f_lo = 100.0;
            nr_options o = options(tol < 1e-6 ? NR_FP64 : NR_FP32);
            o.method = NR_METHOD_CELLRUN;
            nr_plan p = nullptr;
            if (plan(&p, b, tol, o) != NR_OK) return 1;
            std::vector<double> strain(1);
            double power = 0.0;
            fake_hip::launches.clear();
            if (nufft_resample_execute(p, strain.data(), nullptr, &power, nullptr) != NR_OK) return 1;
            bool any = false, all = true;
            for (const fake_hip::Launch& l : fake_hip::launches)
                if (l.is("spread_runs")) {
                    nr::SpreadArgs a;
                    std::memcpy(&a, l.arg.data(), sizeof a);
                    any = true;
                    all = all && (a.rec_stride > 0) == q.rec;
                }
            if (!any || !all) {
                std::printf("%d x %d, %d bins, tol %g: not as expected\n", q.n, (int)q.L, q.K, tol);
                ++bad;
            }
            nufft_resample_destroy(p);
        }
    return bad;
}

// Planning what nodes cannot serve, a segment an instance or a workspace cap far
// below the grids, takes no longer than with the method given: no attempt at nodes
// is carried through and thrown away.
int plan_time()
{
    const int n = 30000;
    Bank own = bank(n, 7680, 256.0, n, 1, 30, 1.0 / 30, 1e-4, 1e-2);
    std::vector<nr_instance> inst;
    for (int i = 0; i < n; ++i) {
        inst.push_back({i, i, 0.0});
        own.segs[i].t_start = 0.0;
    }
    const Bank shared = bank(30, 7680, 256.0, 64, 20, 30, 1.0 / 30);
    int bad = 0;
    for (const bool cap : {false, true}) {
        const Bank& b = cap ? shared : own;
        double best[2] = {1e9, 1e9};
        for (int rep = 0; rep < 7; ++rep)
            for (const int m : {0, 1}) {
                nr_options o = options(NR_FP32);
                o.method = m ? NR_METHOD_CELLRUN : NR_METHOD_AUTO;
                o.max_workspace_bytes = cap ? 3600000 : 0;
                nr_plan p = nullptr;
                const auto t0 = std::chrono::steady_clock::now();
                // (the cap holds neither path: refused after planning on both sides)
                const nr_status st =
                    nufft_resample_plan(&p, b.segs.data(), (int)b.segs.size(), b.tmpls.data(), (int)b.tmpls.size(),
                                        cap ? nullptr : inst.data(), cap ? 0 : n, 1e-6, &o);
                if (st != (cap ? NR_ERR_OUT_OF_MEMORY : NR_OK)) return 1;
                best[m] = std::min(best[m], std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count());
                if (p && has_nodes(p)) return 1;
                nufft_resample_destroy(p);
            }
        std::printf("automatic %.3f s, cell runs %.3f s\n", best[0], best[1]);
        bad += best[0] > 1.35 * best[1];
    }
    return bad;
}

// Templates a segment needs before nodes are planned: both sides of the line.
int worth()
{
    int bad = 0, first[3] = {0, 0, 0};
    const int precision[3] = {NR_FP32, NR_FP64, NR_FP64};
    const double tol[3] = {1e-6, 1e-9, 1e-11};
    for (int k = 0; k < 3; ++k)
        for (int n = 1; n <= 64 && !first[k]; ++n) {
            const Bank b = bank(2, 7680, 256.0, n, 1, 30, 1.0 / 30, 1e-3, 2e-3);
            nr_plan p = nullptr;
            if (plan(&p, b, tol[k], options(precision[k])) != NR_OK) return 1;
            if (has_nodes(p)) first[k] = n;
            nufft_resample_destroy(p);
            // one segment with as many templates as its nodes need is enough, the other has one
            if (first[k]) {
                std::vector<nr_instance> inst;
                for (int i = 0; i < 8 * n; ++i) inst.push_back({0, i % n, 0.0});
                inst.push_back({1, 0, 0.0});
                nr_options o = options(precision[k]);
                p = nullptr;
                if (nufft_resample_plan(&p, b.segs.data(), 2, b.tmpls.data(), n, inst.data(), (int64_t)inst.size(), tol[k],
                                        &o) != NR_OK)
                    return 1;
                bad += !has_nodes(p);
                nufft_resample_destroy(p);
            }
        }
    std::printf("nodes from %d, %d and %d templates a segment on, %d bad\n", first[0], first[1], first[2], bad);
    return bad || !first[0] || !first[1] || !first[2] || first[0] < 2;
}

}  // namespace

int main(int argc, char** argv)
{
    const std::string name = argc > 1 ? argv[1] : "";
    if (name == "strict") return strict();
    if (name == "fallback") return fallback();
    if (name == "full_lds") return full_lds();
    if (name == "large_launches") return large_launches();
    if (name == "tuner") return tuner();
    if (name == "groups") return groups();
    if (name == "copies") return copies();
    if (name == "records") return records();
    if (name == "plan_time") return plan_time();
    if (name == "worth") return worth();
    std::printf("no check of that name\n");
    return 2;
}
