// The life of a context's graphs on the CPU stand-in: what is captured,
// replayed and run kernel by kernel, the limit on their number, and that a
// graph is destroyed only with its context and only when it runs on no
// stream.  The stand-in's calls are wrapped to follow the launches in flight.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <set>
#include <utility>
#include <vector>

#include "spmesl.h"

extern "C" int mock_violations();
extern "C" long mock_launches();
extern "C" long mock_graph_launches();
extern "C" long mock_captures();

static int fails = 0;
static void expect(const char *what, long got, long want)
{
    std::printf("%-64s %ld (want %ld)%s\n", what, got, want, got == want ? "" : "  <-- FAIL");
    if (got != want) ++fails;
}

static std::set<std::pair<hipGraphExec_t, hipStream_t>> in_flight;
static std::set<hipStream_t> gone;
static long destroyed = 0, destroyed_in_flight = 0, waits_on_gone = 0;

extern "C" {
hipError_t __real_hipGraphLaunch(hipGraphExec_t, hipStream_t);
hipError_t __wrap_hipGraphLaunch(hipGraphExec_t ex, hipStream_t s)
{
    in_flight.insert({ex, s});
    return __real_hipGraphLaunch(ex, s);
}
hipError_t __real_hipGraphExecDestroy(hipGraphExec_t);
hipError_t __wrap_hipGraphExecDestroy(hipGraphExec_t ex)
{
    ++destroyed;
    for (const auto &f : in_flight) destroyed_in_flight += f.first == ex;
    return __real_hipGraphExecDestroy(ex);
}
hipError_t __real_hipStreamSynchronize(hipStream_t);
hipError_t __wrap_hipStreamSynchronize(hipStream_t s)
{
    waits_on_gone += (long)gone.count(s);
    for (auto it = in_flight.begin(); it != in_flight.end();) it = it->second == s ? in_flight.erase(it) : ++it;
    return gone.count(s) ? hipSuccess : __real_hipStreamSynchronize(s);
}
hipError_t __real_hipDeviceSynchronize();
hipError_t __wrap_hipDeviceSynchronize()
{
    in_flight.clear();
    return __real_hipDeviceSynchronize();
}
}

struct Case {
    std::vector<double> x, b, om, sig;
    int status = 0;
    spmesl_problem prob{};
    spmesl_result res{};
    spmesl_options opt{};
    Case(int n, int p, int prec) : x((size_t)n * p), b((size_t)p * p), om(b), sig(p)
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
    }
    int async(spmesl_ctx *ctx) { return spmesl_solve_async(ctx, &prob, &opt, &res, &status); }
};

struct Counts {
    long k = mock_launches(), c = mock_captures(), g = mock_graph_launches();
};
// kernel by kernel: no graph work; capture: captured and launched; replay:
// launched alone
template <typename F> static void run_as(const char *what, int how, F call)
{
    const Counts a;
    expect(what, call(), SPMESL_OK);
    const Counts b;
    expect("  captures", b.c - a.c, how == 1);
    expect("  graph launches", b.g - a.g, how != 0);
    expect("  kernels enqueued", b.k > a.k, how != 2);
}
enum { kByKernel = 0, kCapture = 1, kReplay = 2 };

int main()
{
    spmesl_ctx *ctx = nullptr;
    expect("create", spmesl_create(&ctx, 0, nullptr), SPMESL_OK);
    // every entry point: kernel by kernel, captured, replayed, replayed
    for (int prec : {SPMESL_FP64, SPMESL_FP32, SPMESL_MIXED}) {
        Case a(40, 60, prec), b(30, 90, prec);
        const int how[4] = {kByKernel, kCapture, kReplay, kReplay};
        for (int h : how) run_as("solve", h, [&] { return spmesl_solve(ctx, &a.prob, &a.opt, &a.res); });
        for (int h : how) run_as("async", h, [&] { return a.async(ctx); });
        spmesl_problem ps[2] = {a.prob, b.prob};
        spmesl_result rs[2] = {a.res, b.res};
        int st[2];
        // (a batch's tables are uploaded each time; the first call may grow the workspace)
        for (int h : how) run_as("batch", h, [&] { return spmesl_solve_batch(ctx, 2, ps, &a.opt, nullptr, rs, st); });
        a.opt.flags = SPMESL_FLAG_EAGER;
        for (int i = 0; i < 3; ++i) run_as("eager", kByKernel, [&] { return a.async(ctx); });
    }
    expect("graphs destroyed so far", destroyed, 0);
    spmesl_destroy(ctx);
    expect("graphs destroyed with the context", destroyed, 9);

    // cycles: five distinct calls never repeat one of the last four; four do
    expect("create", spmesl_create(&ctx, 0, nullptr), SPMESL_OK);
    Case c(40, 60, SPMESL_FP64);
    for (int len : {5, 4}) {
        for (int round = 0; round < 3; ++round)
            for (int i = 0; i < len; ++i) {
                c.opt.lambda0 = 0.1 * len + 0.01 * i;
                run_as("call of a cycle", len == 5 || round == 0 ? kByKernel : (round == 1 ? kCapture : kReplay),
                       [&] { return c.async(ctx); });
            }
    }
    // the limit: 64 graphs, then kernel by kernel, and the held ones still replay
    int held = 4;
    for (int i = 0; i < 70; ++i) {
        c.opt.lambda0 = 1.0 + 0.01 * i;
        run_as("first call", kByKernel, [&] { return c.async(ctx); });
        run_as("its repeat", held < 64 ? kCapture : kByKernel, [&] { return c.async(ctx); });
        run_as("its second repeat", held < 64 ? kReplay : kByKernel, [&] { return c.async(ctx); });
        if (held < 64) ++held;
    }
    c.opt.lambda0 = 1.0;
    run_as("a call held from before", kReplay, [&] { return c.async(ctx); });
    destroyed = 0;
    spmesl_destroy(ctx);
    expect("graphs destroyed with the context", destroyed, 64);
    expect("... none of them in flight", destroyed_in_flight, 0);

    // a graph in flight on a stream that the context has left (and that may be
    // gone itself) when the context is destroyed
    for (const bool stream_gone : {false, true}) {
        hipStream_t s1, s2;
        hipStreamCreateWithFlags(&s1, hipStreamNonBlocking);
        hipStreamCreateWithFlags(&s2, hipStreamNonBlocking);
        expect("create", spmesl_create(&ctx, 0, s1), SPMESL_OK);
        Case d(40, 60, SPMESL_MIXED);
        for (int i = 0; i < 3; ++i) expect("async on one stream", d.async(ctx), SPMESL_OK);
        spmesl_set_stream(ctx, s2);
        expect("async on another", d.async(ctx), SPMESL_OK);
        if (stream_gone) gone.insert(s1);
        spmesl_destroy(ctx);
        expect("graphs destroyed in flight", destroyed_in_flight, 0);
        expect("waits on a stream that is gone", waits_on_gone, 0);
        gone.clear();
        hipStreamDestroy(s1);
        hipStreamDestroy(s2);
    }
    expect("rule violations", mock_violations(), 0);
    std::printf("graphs: %d failed\n", fails);
    return fails ? 1 : 0;
}
