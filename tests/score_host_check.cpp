// The device code of csrc/rv.hip on the CPU (tests/emulator; the test that builds this
// passes its device half as RV_DEVICE_SOURCE): the scoring of a large cluster under
// many orders of its workgroup's waves, against the count of every hypothesis; the refit
// by one wave, four and sixteen.
//   score_host_check no-reference | other-workgroups | refit-order | deferred
#include <algorithm>

#include RV_DEVICE_SOURCE

namespace {

struct Cluster {
    std::vector<float> theta, vd;
    std::vector<StagedPoint> staged;
    std::vector<StagedLow> low;
    Points pts;
    Span sp;
    void stage() {
        staged.resize(theta.size());
        low.resize(theta.size());
        for (size_t p = 0; p < theta.size(); ++p)
            stage_point(theta.data(), vd.data(), (int64_t)p, Staging{staged.data(), low.data()});
        pts = {staged.data(), low.data(), theta.data()};
        sp = {0, (int64_t)theta.size(), true};
    }
};

Cluster make_cluster(int n, uint32_t seed, double outliers, double finite) {
    std::mt19937 rng(seed);
    std::uniform_real_distribution<double> u(0, 1);
    std::normal_distribution<double> g(0, 0.05);
    Cluster c;
    for (int i = 0; i < n; ++i) {
        const double t = 2 * u(rng) - 1;
        double v = 12 * cos(t) - 7 * sin(t) + g(rng);
        if (u(rng) < outliers) v = 80 * u(rng) - 40;
        c.theta.push_back((float)t);
        c.vd.push_back(u(rng) < finite ? (float)v : NAN);
    }
    c.stage();
    return c;
}

constexpr float kTau = 0.15f;

// Count of hypothesis h as the rows form makes it, -1 for an invalid one.
int64_t count_of(const Cluster &c, ClusterId id, uint32_t h) {
    const Hypothesis y = make_hypothesis(c.pts, c.sp, h, id.local, id.key0, id.key1);
    const float hx = (float)y.vx, hy = (float)y.vy;
    if (std::isnan(hx)) return -1;
    int64_t n = 0;
    for (const StagedPoint &q : c.staged)
        n += fabsf(fmaf(-hy, q.s, fmaf(-hx, q.c, q.v))) < kTau ? 1 : 0;
    return n;
}

unsigned long long full_key(const Cluster &c, ClusterId id, int64_t first, int nh) {
    unsigned long long best = 0;
    for (int64_t h = first; h < first + nh; ++h) {
        const int64_t n = count_of(c, id, (uint32_t)h);
        if (n >= 0 && hyp_key((uint32_t)n, h) > best) best = hyp_key((uint32_t)n, h);
    }
    return best;
}

ClusterId cluster_id(uint32_t seed) { return {0, 3, seed, 77}; }

ScoreShared<kScoreBlock> shared;

template <bool kHalf>
unsigned long long pruned(const Cluster &c, ClusterId id, int64_t first, int nh, uint32_t order,
                          unsigned long long *best_key) {
    unsigned long long keys[kScoreBlock];
    memset((void *)&shared, 0xFF, sizeof shared);  // what an earlier workgroup left: NaN, -1
    emu::run(kScoreBlock, order, [&] {
        const uint32_t t = threadIdx.x;
        const unsigned long long k = score_hypotheses<kScoreBlock, kPassRows, kHalf>(
            c.sp, id, first, nh, (int32_t)first + nh, c.pts, kTau, kRowsMax, 0, 0, 0, kHalf, false, shared,
            best_key, nullptr);
        keys[t] = k;
    });
    for (int t = 1; t < kScoreBlock; ++t)
        if (keys[t] != keys[0]) emu::fail("the threads' keys differ, thread, order", t, (int)order);
    return keys[0];
}

void check(bool ok, const char *what, int a, int b) {
    if (!ok) emu::fail(what, a, b);
}

// No usable hypothesis among the workgroup's first 64 (one point in a dozen is
// finite), a few after them.
void no_reference() {
    int cases = 0;
    for (uint32_t seed = 0; cases < 12; ++seed) {
        const Cluster c = make_cluster(330 + (int)seed % 90, seed, 0.2, 0.08);
        const ClusterId id = cluster_id(seed);
        const int64_t first = seed % 2 ? 512 : 0;
        const int nh = seed % 3 ? 256 : 700;
        bool usable = false;
        for (int h = 0; h < kWave; ++h) usable |= count_of(c, id, (uint32_t)(first + h)) >= 0;
        const unsigned long long want = full_key(c, id, first, nh);
        if (usable || want == 0) continue;
        ++cases;
        for (uint32_t order = 0; order < 12; ++order)
            check(pruned<false>(c, id, first, nh, order, nullptr) == want,
                  "no reference: wrong key, seed, order", (int)seed, (int)order);
    }
}

// Another workgroup of the cluster merges a key just below this one's best after some
// of the waves have read the cluster's, before the others do.
template <bool kHalf>
void other_workgroups() {
    for (uint32_t seed = 0; seed < 8; ++seed) {
        const Cluster c = make_cluster(700 + 37 * (int)seed, 100 + seed, 0.35, 1.0);
        const ClusterId id = cluster_id(seed);
        const unsigned long long want = full_key(c, id, 256, 256);
        for (uint32_t order = 0; order < 24; ++order) {
            unsigned long long best_key = 0;
            uint32_t loads = 0;
            emu::on_load = [&] {
                if (loads++ == (order % 4) * kWave) best_key = want - 1;
            };
            const unsigned long long got = pruned<kHalf>(c, id, 256, 256, order, &best_key);
            emu::on_load = nullptr;
            check(loads > 0, "no load of the cluster's key", (int)seed, (int)order);
            check(got == want, kHalf ? "FP16 form: winner lost, seed, order"
                                     : "winner lost, seed, order", (int)seed, (int)order);
        }
    }
}

struct Refit {
    float vx, vy, heading;
    int32_t n_inliers, n_near;
    uint8_t status;
    uint32_t bits[512];
};

// The cluster's refit by `waves` waves of a workgroup of kWaves, its points from `at` on.
template <int kWaves>
Refit refit(const Cluster &c, int waves, int64_t at, uint32_t order) {
    static RefitShared<kWaves> sh;
    memset((void *)&sh, 0xFF, sizeof sh);
    std::vector<StagedPoint> staged(at, {NAN, NAN, NAN});
    std::vector<StagedLow> low(at, {NAN, NAN});
    std::vector<float> theta(at, NAN);
    staged.insert(staged.end(), c.staged.begin(), c.staged.end());
    low.insert(low.end(), c.low.begin(), c.low.end());
    theta.insert(theta.end(), c.theta.begin(), c.theta.end());
    const Points pts = {staged.data(), low.data(), theta.data()};
    const Span sp = {at, c.sp.n, true};
    const ClusterId id = cluster_id(5);
    unsigned long long best = 0;
    for (uint32_t h = 0; h < 64 && best == 0; ++h)
        if (count_of(c, id, h) >= 0) best = hyp_key(1, h);
    check(best != 0, "no valid pair, points", (int)c.sp.n, 0);
    Refit r;
    memset(&r, 0, sizeof r);
    const Outputs o = {&r.vx, &r.vy, &r.heading, &r.n_inliers, &r.status, &r.n_near, nullptr,
                       nullptr, at + c.sp.n <= 512 * 32 ? r.bits : nullptr};
    emu::run(waves * kWave, order, [&] {
        refit_cluster<kWaves>(sp, id, best, pts, 1.0f, o, (int)threadIdx.x / kWave, waves, sh);
    });
    return r;
}

// Nearly all points share one azimuth, so that another order of the sums shows.
void refit_order() {
    for (int n : {2, 63, 64, 65, 130, 255, 256, 257, 700, 1023, 1024, 1025, 4097, 8191, 8192, 9001}) {
        std::mt19937 rng(n);
        std::normal_distribution<double> g(0, 1);
        Cluster c;
        for (int i = 0; i < n; ++i) {
            const double t = 0.3 + 1e-6 * g(rng) + (i % 3 == 1 ? 1.5e-3 : 0.0);
            c.theta.push_back((float)t);
            c.vd.push_back((float)(9 * cos(t) - 4 * sin(t) + 0.05 * g(rng)));
        }
        c.stage();
        const Refit want = refit<4>(c, 4, 0, 1);
        check(want.n_inliers > n / 2, "few inliers, points", n, want.n_inliers);
        const auto same = [&](const Refit &r, int64_t at, int waves) {
            check(!memcmp(&r, &want, offsetof(Refit, bits)), "refit differs, points, waves", n, waves);
            if (at + n <= 512 * 32)
                for (int i = 0; i < n; ++i)
                    check(((r.bits[(at + i) / 32] >> ((at + i) % 32)) & 1) ==
                              ((want.bits[i / 32] >> (i % 32)) & 1),
                          "mask differs, points, waves", n, waves);
        };
        for (int64_t at : {0, 1, 31, 77}) {
            same(refit<4>(c, 4, at, 2), at, 4);
            same(refit<16>(c, 16, at, 3), at, 16);
            if (n < kRefitBigPoints) same(refit<4>(c, 1, at, 4), at, 1);
        }
    }
}

// A refit kernel over clusters of which some are deferred, its workgroups one after the
// other in a drawn order, against the refit of the full count's key.
template <int B>
void deferred(int32_t n_hyp, uint32_t seed) {
    std::mt19937 rng(seed);
    std::vector<Cluster> clusters;
    for (int n : {9000, 4200, 2050, 1500, 1024, 1023, 300, 64, 2, 1})
        clusters.push_back(make_cluster(n, seed * 31 + n, 0.8, n == 2050 ? 0.0 : 1.0));
    const int64_t K = (int64_t)clusters.size();
    Cluster all;
    std::vector<int32_t> off(1, 0), order;
    for (const Cluster &c : clusters) {
        all.theta.insert(all.theta.end(), c.theta.begin(), c.theta.end());
        all.vd.insert(all.vd.end(), c.vd.begin(), c.vd.end());
        off.push_back((int32_t)all.theta.size());
        order.push_back((int32_t)order.size());
    }
    all.stage();
    const int64_t n_big[2] = {5, 0};  // of kRefitBigPoints points or more, in the order
    std::vector<Refit> got(K);
    std::vector<float> vx(K), vy(K), heading(K);
    std::vector<int32_t> n_inliers(K), n_near(K), best_hyp(K);
    std::vector<uint8_t> status(K);
    std::vector<uint32_t> bits(all.theta.size() / 32 + 1);
    const Outputs o = {vx.data(), vy.data(), heading.data(), n_inliers.data(), status.data(),
                       n_near.data(), best_hyp.data(), nullptr, bits.data()};
    std::vector<unsigned long long> keys(K), want(K);
    const FrameClusterAt at = {off.data(), order.data(), (int64_t)all.theta.size(), seed, 3, 0, 0,
                               keys.data()};
    int n_deferred = 0;
    for (int64_t k = 0; k < K; ++k) {
        const Span sp = at.span(k);
        const ClusterId id = at.id(k);
        Cluster c = clusters[k];
        want[k] = sp.n < 2 ? 0 : full_key(c, id, 0, n_hyp);
        const bool defer = sp.n >= kRefitBigPoints && (k < 3 || rng() % 2);
        n_deferred += defer;
        keys[k] = defer ? kDeferred | (rng() % 2 ? want[k] & ~1ull : 0) : want[k];
    }
    const auto run = [&](const std::vector<uint32_t> &blocks, uint32_t grid) {
        gridDim.x = grid;
        for (uint32_t b : blocks) {
            blockIdx.x = b;
            static RefitSpace<B> space;
            memset((void *)&space, 0xFF, sizeof space);
            emu::run(B, rng(), [&] {
                refit_planned<B>(K, n_big, at, n_hyp, all.pts, 1.0f * kTau, o, space, kNoneDone);
            });
        }
    };
    const uint32_t extra = 8 * (1 + rng() % 3);
    std::vector<uint32_t> blocks(K + extra);
    for (uint32_t b = 0; b < blocks.size(); ++b) blocks[b] = b;
    std::shuffle(blocks.begin(), blocks.end(), rng);
    run(blocks, (uint32_t)blocks.size());
    const auto vx1 = vx, vy1 = vy, heading1 = heading;
    const auto n1 = n_inliers, near1 = n_near, best1 = best_hyp;
    const auto status1 = status;
    const auto bits1 = bits;
    keys = want;
    for (int64_t k = 0; k < K; ++k) order[k] = (int32_t)k;
    std::fill(bits.begin(), bits.end(), 0);
    std::fill(status.begin(), status.end(), 99);
    blocks.resize(K);
    for (uint32_t b = 0; b < blocks.size(); ++b) blocks[b] = b;
    run(blocks, (uint32_t)K);
    const auto same = [&](const void *a, const void *b, size_t n, const char *what) {
        check(!memcmp(a, b, n), what, (int)seed, n_deferred);
    };
    same(vx1.data(), vx.data(), K * 4, "deferred: vx, seed, deferred clusters");
    same(vy1.data(), vy.data(), K * 4, "deferred: vy, seed, deferred clusters");
    same(heading1.data(), heading.data(), K * 4, "deferred: heading, seed, deferred clusters");
    same(n1.data(), n_inliers.data(), K * 4, "deferred: n_inliers, seed, deferred clusters");
    same(near1.data(), n_near.data(), K * 4, "deferred: n_near, seed, deferred clusters");
    same(best1.data(), best_hyp.data(), K * 4, "deferred: best, seed, deferred clusters");
    same(status1.data(), status.data(), K, "deferred: status, seed, deferred clusters");
    same(bits1.data(), bits.data(), bits.size() * 4, "deferred: mask, seed, deferred clusters");
}

}  // namespace

int main(int argc, char **argv) {
    const char *what = argc > 1 ? argv[1] : "";
    if (!strcmp(what, "no-reference")) {
        no_reference();
    } else if (!strcmp(what, "other-workgroups")) {
        other_workgroups<false>();
        other_workgroups<true>();
    } else if (!strcmp(what, "refit-order")) {
        refit_order();
    } else if (!strcmp(what, "deferred")) {
        for (uint32_t seed = 0; seed < 3; ++seed) deferred<kLongBlock>(seed % 2 ? 512 : 257, seed + 50);
    } else {
        return 2;
    }
    printf("ok\n");
    return 0;
}
