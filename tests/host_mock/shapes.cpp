// Launch shapes and the autotuner on the CPU stand-in: where the outputs are
// cleared follows from fill_split alone, and the autotuner returns the
// defaults unless repeated calls are faster with what it found.  Kernels are
// counted (a fill on the second stream is a launch of its own); the times the
// autotuner reads are scripted here (hipEventElapsedTime is wrapped).
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstring>
#include <vector>

#include "spmesl.h"

extern "C" long mock_launches();
extern "C" long mock_graph_launches();

static int fails = 0;
static void expect(const char *what, long got, long want)
{
    std::printf("%-64s %ld (want %ld)%s\n", what, got, want, got == want ? "" : "  <-- FAIL");
    if (got != want) ++fails;
}

// a time per elapsed-time query: `eager` when no graph was launched since the
// last query (each query a twentieth less), else `replay` of the query's rank
static double eager_ms = 1.0;
static std::vector<double> replay_ms;
static size_t replay_at = 0;
static long graphs_seen = 0;
extern "C" hipError_t __wrap_hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t)
{
    const long g = mock_graph_launches();
    if (g == graphs_seen) {
        *ms = (float)eager_ms;
        eager_ms *= 0.95;
    } else {
        *ms = (float)(replay_at < replay_ms.size() ? replay_ms[replay_at] : 1.0);
        ++replay_at;
    }
    graphs_seen = g;
    return hipSuccess;
}

struct Case {
    int p, prec;
    std::vector<double> x, b, om, sig;
    spmesl_problem prob{};
    spmesl_result res{};
    spmesl_options opt{};
    Case(int n, int p_, int prec_) : p(p_), prec(prec_), x((size_t)n * p_), b((size_t)p_ * p_), om(b), sig(p_)
    {
        prob.X = x.data();
        prob.n = n;
        prob.p = p;
        prob.ldx = p;
        res.B = b.data();
        res.sigma = sig.data();
        res.Omega = om.data();
        opt.lambda0 = 0.3;
        opt.tol = 1e-8;
        opt.precision = prec;
        opt.flags = SPMESL_FLAG_EAGER;
    }
    long launches(spmesl_ctx *ctx, const spmesl_tuning *t)
    {
        expect("set_tuning", spmesl_set_tuning(ctx, t), SPMESL_OK);
        const long l0 = mock_launches();
        expect("solve", spmesl_solve(ctx, &prob, &opt, &res), SPMESL_OK);
        return mock_launches() - l0;
    }
};

int main()
{
    spmesl_ctx *ctx = nullptr;
    expect("create", spmesl_create(&ctx, 0, nullptr), SPMESL_OK);
    for (int prec : {SPMESL_FP64, SPMESL_FP32, SPMESL_MIXED}) {
        Case c(40, 300, prec);
        const long def = c.launches(ctx, nullptr);
        // a field that is not the placement leaves the placement alone
        for (int field = 0; field < 4; ++field) {
            spmesl_tuning t{};
            (field == 0 ? t.dense_block : field == 1 ? t.fill_blocks : field == 2 ? t.kkt_rows : t.screen_permille) =
                field == 2 ? 1 : 64;
            expect("launches with one other field set", c.launches(ctx, &t), def);
        }
        for (int split : {1, 2}) {  // two fills on the second stream
            spmesl_tuning t{};
            t.fill_split = split;
            expect("launches with the placement set", c.launches(ctx, &t), def + 2);
        }
        spmesl_tuning bad{};
        bad.fill_split = 3;
        expect("fill_split 3 is refused", spmesl_set_tuning(ctx, &bad), SPMESL_EINVAL);
        expect("reset", spmesl_set_tuning(ctx, nullptr), SPMESL_OK);
        // the autotuner: every candidate looks faster kernel by kernel
        //; replays decide
        for (const bool faster : {false, true}) {
            spmesl_ctx *fresh = nullptr;
            expect("create", spmesl_create(&fresh, 0, nullptr), SPMESL_OK);
            eager_ms = 1.0;
            replay_at = 0;
            // (three runs of the defaults, then of what was found)
            replay_ms = {1.0, 1.0, 1.0};
            for (int i = 0; i < 3; ++i) replay_ms.push_back(faster ? 0.5 : 1.0);
            // the untimed first two calls query as well: the capture of each
            // launches its graph once
            replay_ms.insert(replay_ms.begin(), 9.0);
            replay_ms.insert(replay_ms.begin() + 4, 9.0);
            graphs_seen = mock_graph_launches();
            spmesl_tuning best{};
            double ms = 0.0;
            spmesl_options o = c.opt;
            o.flags = 0;
            expect("autotune", spmesl_autotune(fresh, &c.prob, &o, &c.res, 4, &best, &ms), SPMESL_OK);
            spmesl_tuning now{};
            expect("get_tuning", spmesl_get_tuning(fresh, &now), SPMESL_OK);
            expect("the context holds what was returned", std::memcmp(&now, &best, sizeof now), 0);
            const bool is_def = best.dense_block == 64 && best.fill_blocks == 64 && best.screen_permille == 800 &&
                                best.fill_split == 0 && best.kkt_rows == 4;
            expect(faster ? "faster when replayed: kept" : "not faster when replayed: the defaults", is_def, !faster);
            expect("milliseconds of the shapes returned, in 1e-6", (long)(ms * 1e6 + 0.5), faster ? 125000 : 250000);
            const long l0 = mock_launches();
            expect("solve", spmesl_solve(fresh, &c.prob, &c.opt, &c.res), SPMESL_OK);
            if (!faster) expect("launches of a tuned context's solve", mock_launches() - l0, def);
            spmesl_destroy(fresh);
        }
    }
    spmesl_destroy(ctx);
    std::printf("launch shapes: %d failed\n", fails);
    return fails ? 1 : 0;
}
