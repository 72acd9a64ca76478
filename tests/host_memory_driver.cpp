// Plans and chains where device memory runs out (tests/test_memory_limits_host.py): a choice of kernel that needs weights in a form of its own gives
// way to one that reads them as they are.  Runs against fake_hip_runtime.hpp.
#include "fake_hip_runtime.hpp"
#include "mnn_conv.h"

#include <sys/wait.h>
#include <unistd.h>

#include <cstdio>
#include <functional>
#include <string>

namespace {

int failures = 0;
#define CHECK(cond) \
    do { if (!(cond)) { std::printf("line %d: %s   [%s]\n", __LINE__, #cond, mnn_last_error()); ++failures; } } while (0)

struct LayerSpec { mnn_conv_shape s; mnn_conv_geom g; mnn_conv_options o; size_t other_form, plain; const char* kernel; };

float* some(size_t i) { return reinterpret_cast<float*>((uintptr_t)0x10000 * (i + 1)); }

mnn_conv_options options(int kind, int tile, int prec)
{
    mnn_conv_options o;
    mnn_conv_options_default(&o);
    o.force_kind = kind;
    o.force_prec = prec;
    if (kind == MNN_SCHEME_WINOGRAD) { o.force_tile_n = tile; o.force_variant = MNN_WINO_UNFUSED; }
    return o;
}

size_t parts(int k, int c, int taps, int np) { return (size_t)((k + 127) / 128 * 128) * ((c + 15) / 16 * 16) * taps * 2 * np; }

std::string described(mnn_conv_plan_t p)
{
    char buf[256];
    mnn_conv_plan_describe(p, buf, sizeof buf);
    return buf;
}

// the plan, what it says of itself, and whether a pass runs the kernel; the plan is freed
struct Outcome { int rc; std::string name; size_t bytes; bool runs_kernel; };
Outcome plan_and_run(const LayerSpec& l)
{
    mnn_conv_plan_t p = nullptr;
    Outcome o{mnn_conv_plan(&l.s, &l.g, &l.o, nullptr, &p), "", 0, false};
    if (o.rc) return o;
    o.name = described(p);
    o.bytes = mnn_conv_workspace_bytes(p);
    fake::launched.clear();
    CHECK(mnn_conv_run(p, some(0), some(1), some(2), some(3), nullptr) == MNN_OK);
    o.runs_kernel = fake::ran(l.kernel);
    mnn_conv_plan_destroy(p);
    return o;
}

// In a process of its own, which starts with no choices: true if all checks passed.
bool in_child(const std::function<void()>& f)
{
    std::fflush(stdout);
    const pid_t pid = fork();
    if (pid == 0) {
        failures = 0;
        f();
        std::fflush(stdout);
        _exit(failures ? 1 : 0);
    }
    int status = 1;
    return pid > 0 && waitpid(pid, &status, 0) == pid && status == 0;
}

void check_layer(const char* what, const LayerSpec& l)
{
    const char* const file = "choices.txt";
    const bool beside = l.o.force_kind == MNN_SCHEME_WINOGRAD;       // the other form lies beside U, or in its place
    auto plenty = [](size_t) { return false; };
    auto scarce = [&](size_t bytes) { return bytes == l.other_form; };
    fake::takes = [&](const std::string& k) { return k.find(l.kernel) != std::string::npos ? 0.1f : 1.f; };

    // a remembered choice, and no room for its weights
    auto remembered = [&](const std::string& chosen) {
        fake::refuse = scarce;
        const Outcome poor = plan_and_run(l);
        CHECK(poor.rc == MNN_OK && !poor.runs_kernel && poor.bytes == l.plain && poor.name != chosen);
        mnn_chain_layer cl{};
        cl.shape = l.s; cl.geom = l.g;
        mnn_chain_t ch = nullptr;
        CHECK(mnn_chain_create(&cl, 1, &l.o, nullptr, &ch) == MNN_OK);
        if (ch) {
            CHECK(mnn_chain_set_weights(ch, 0, some(1), some(2), nullptr) == MNN_OK);
            fake::launched.clear();
            CHECK(mnn_chain_run(ch, some(0), some(3), nullptr) == MNN_OK && !fake::ran(l.kernel));
            mnn_chain_destroy(ch);
        }
        fake::refuse = plenty;
        const Outcome again = plan_and_run(l);                       // the choice itself is still remembered
        CHECK(again.runs_kernel && again.name == chosen);
        CHECK(fake::live.empty());
    };
    bool ok = in_child([&] {
        const Outcome rich = plan_and_run(l);
        CHECK(rich.rc == MNN_OK && rich.runs_kernel && rich.bytes == (beside ? l.plain + l.other_form : l.other_form));
        CHECK(mnn_conv_cache_save(file) == MNN_OK);
        remembered(rich.name);
    });
    ok &= in_child([&] {
        CHECK(mnn_conv_cache_load(file) == MNN_OK);
        const std::string chosen = plan_and_run(l).name;
        remembered(chosen);
    });
    // timed while there was no room for the other form: good for a chain, which times nothing, but not for good, and not for a file
    ok &= in_child([&] {
        fake::refuse = scarce;
        const Outcome poor = plan_and_run(l);
        CHECK(poor.rc == MNN_OK && !poor.runs_kernel);
        CHECK(mnn_conv_cache_save("poor.txt") == MNN_OK);
        mnn_chain_layer cl{};
        cl.shape = l.s; cl.geom = l.g;
        mnn_chain_t ch = nullptr;
        CHECK(mnn_chain_create(&cl, 1, &l.o, nullptr, &ch) == MNN_OK);
        if (ch) {
            char buf[256] = "";
            mnn_chain_layer_describe(ch, 0, buf, sizeof buf);
            CHECK(poor.name == buf);
            mnn_chain_destroy(ch);
        }
        fake::refuse = plenty;
        CHECK(plan_and_run(l).runs_kernel);
        CHECK(fake::live.empty());
    });
    ok &= in_child([&] {
        CHECK(mnn_conv_cache_load("poor.txt") == MNN_OK);
        CHECK(plan_and_run(l).runs_kernel);
    });
    std::printf("%s: %s\n", what, ok ? "ok" : "FAILED");
    failures += !ok;
}

mnn_conv_shape shape(int n, int c, int h, int w, int k, int ks) { return mnn_conv_shape{n, c, h, w, k, ks, ks}; }
mnn_conv_geom geom(int stride, int pad) { return mnn_conv_geom{stride, stride, pad, pad, 1, 1}; }

// The products at the bottom of two Strassen levels have the shape of F(3,5)'s 49, but no weights as parts: they are timed on their own.
void check_strassen_beside_winograd()
{
    bool ok = in_child([] {
        fake::takes = [](const std::string& k) { return k.find("gemm_prepared") != std::string::npos ? 0.1f : 1.f; };
        const LayerSpec l{shape(8, 64, 21, 21, 96, 5), geom(1, 2), options(MNN_SCHEME_WINOGRAD, 3, MNN_GEMM_FP32), 0, 0, "gemm_prepared"};
        CHECK(plan_and_run(l).runs_kernel);
        mnn_gemm_desc d{};
        d.M = 4 * 96; d.R = 4 * 64; d.ncols = d.L = 4 * 392; d.batch = 1; d.lda = d.M;
        d.strideB_row = d.strideD_row = d.ncols;
        mnn_strassen_t h = nullptr;
        fake::launched.clear();
        CHECK(mnn_strassen_create(&d, 2, nullptr, &h) == MNN_OK);
        CHECK(fake::ran("gemm_split_kernel") && !fake::ran("gemm_prepared"));
        mnn_strassen_destroy(h);
        CHECK(plan_and_run(l).runs_kernel);
        CHECK(fake::live.empty());
    });
    // on its own it is remembered and saved like any other
    mnn_gemm_desc d{};
    d.M = d.R = d.ncols = d.L = d.lda = 512; d.batch = 1;
    d.strideB_row = d.strideD_row = d.ncols;
    auto create = [&](int levels) {
        mnn_strassen_t h = nullptr;
        fake::launched.clear();
        CHECK(mnn_strassen_create(&d, levels, nullptr, &h) == MNN_OK);
        mnn_strassen_destroy(h);
        return fake::ran("gemm_");
    };
    ok &= in_child([&] {
        CHECK(create(0) && create(1));
        CHECK(!create(0) && !create(1));
        CHECK(mnn_conv_cache_save("strassen.txt") == MNN_OK);
    });
    ok &= in_child([&] {
        CHECK(mnn_conv_cache_load("strassen.txt") == MNN_OK);
        CHECK(!create(0) && !create(1));
    });
    std::printf("Strassen beside Winograd: %s\n", ok ? "ok" : "FAILED");
    failures += !ok;
}

// Launching runs out of host memory: every entry point that launches says so, none lets the exception out, and the next call works.
void check_exceptions()
{
    const bool ok = in_child([] {
        fake::takes = [](const std::string&) { return 1.f; };
        const LayerSpec layers[] = {{shape(2, 64, 28, 28, 96, 3), geom(1, 1), options(MNN_SCHEME_WINOGRAD, 4, MNN_GEMM_FP32), 0, 0, ""},
                                    {shape(2, 64, 28, 28, 96, 1), geom(1, 0), options(MNN_SCHEME_GEMM1X1, 0, MNN_GEMM_FP32), 0, 0, ""},
                                    {shape(2, 64, 28, 28, 96, 3), geom(2, 1), options(MNN_SCHEME_DIRECT, 0, MNN_GEMM_FP32), 0, 0, ""}};
        for (const LayerSpec& l : layers) {
            mnn_conv_plan_t p = nullptr;
            CHECK(mnn_conv_plan(&l.s, &l.g, &l.o, nullptr, &p) == MNN_OK);
            mnn_chain_layer cl{};
            cl.shape = l.s; cl.geom = l.g;
            mnn_chain_t ch = nullptr;
            CHECK(mnn_chain_create(&cl, 1, &l.o, nullptr, &ch) == MNN_OK && mnn_chain_set_weights(ch, 0, some(1), nullptr, nullptr) == MNN_OK);
            float ms[MNN_STAGE_COUNT];
            fake::launch_throws = true;
            CHECK(mnn_conv_run(p, some(0), some(1), some(2), some(3), nullptr) == MNN_E_OOM);
            CHECK(mnn_conv_run_stage(p, MNN_STAGE_GEMM, some(0), some(1), some(2), some(3), nullptr) == MNN_E_OOM);
            CHECK(mnn_conv_run_timed(p, some(0), some(1), some(2), some(3), nullptr, 1, ms) == MNN_E_OOM);
            CHECK(mnn_conv_set_weights(p, some(1), nullptr) == MNN_E_OOM);
            CHECK(mnn_chain_run(ch, some(0), some(3), nullptr) == MNN_E_OOM);
            CHECK(mnn_chain_set_weights(ch, 0, some(1), nullptr, nullptr) == MNN_E_OOM);
            CHECK(mnn_conv_run_static(&l.s, &l.g, l.o.force_tile_n, some(0), some(1), some(2), some(3), nullptr) == MNN_E_OOM);
            fake::launch_throws = false;
            fake::pushed.clear();
            CHECK(mnn_conv_run(p, some(0), some(1), some(2), some(3), nullptr) == MNN_OK && mnn_chain_run(ch, some(0), some(3), nullptr) == MNN_OK);
            mnn_conv_plan_destroy(p);
            mnn_chain_destroy(ch);
        }
        mnn_gemm_desc d{};
        d.M = d.R = d.ncols = d.L = d.lda = 256; d.batch = 1;
        d.strideB_row = d.strideD_row = 256;
        mnn_strassen_t h = nullptr;
        CHECK(mnn_strassen_create(&d, 1, nullptr, &h) == MNN_OK && mnn_strassen_set_left(h, some(1), nullptr) == MNN_OK);
        fake::launch_throws = true;
        CHECK(mnn_gemm_f32(&d, some(0), some(1), nullptr, some(2), nullptr) == MNN_E_OOM);
        CHECK(mnn_strassen_set_left(h, some(1), nullptr) == MNN_E_OOM && mnn_strassen_run(h, some(0), nullptr, some(2), nullptr) == MNN_E_OOM);
        fake::launch_throws = false;
        mnn_strassen_destroy(h);
        CHECK(fake::live.empty());
    });
    std::printf("exceptions: %s\n", ok ? "ok" : "FAILED");
    failures += !ok;
}

// A form of the weights that no configuration worth timing reads is not made for timing either.
void check_forms_made()
{
    struct Case { const char* what; LayerSpec l; bool made; };
    const Case cases[] = {
        {"pointwise, result of 103 MB", {shape(32, 256, 28, 28, 1024, 1), geom(1, 0), options(MNN_SCHEME_GEMM1X1, 0, MNN_GEMM_FP32), parts(1024, 256, 1, 3), 0, ""}, false},
        {"pointwise, result of 6 MB", {shape(8, 256, 28, 28, 256, 1), geom(1, 0), options(MNN_SCHEME_GEMM1X1, 0, MNN_GEMM_FP32), parts(256, 256, 1, 3), 0, ""}, true},
        {"Winograd, result of 460 MB", {shape(16, 128, 128, 128, 128, 3), geom(1, 1), options(MNN_SCHEME_WINOGRAD, 4, MNN_GEMM_FP32), 36 * parts(128, 128, 1, 3), 0, ""}, false},
        {"Winograd, result of 7 MB", {shape(8, 128, 28, 28, 128, 3), geom(1, 1), options(MNN_SCHEME_WINOGRAD, 4, MNN_GEMM_FP32), 36 * parts(128, 128, 1, 3), 0, ""}, true},
        {"sliding window, operand order, 1568 tiles", {shape(32, 66, 56, 56, 64, 3), geom(1, 1), options(MNN_SCHEME_DIRECT, 0, MNN_GEMM_FP32), (size_t)4 * 3 * 9 * 2048, 0, ""}, false},
        {"sliding window, operand order, 1568 tiles of 32 channels", {shape(32, 66, 56, 56, 32, 3), geom(1, 1), options(MNN_SCHEME_DIRECT, 0, MNN_GEMM_FP32), (size_t)2 * 3 * 9 * 2048, 0, ""}, true},
        {"sliding window, operand order, 49 tiles", {shape(1, 66, 56, 56, 64, 3), geom(1, 1), options(MNN_SCHEME_DIRECT, 0, MNN_GEMM_FP32), (size_t)4 * 3 * 9 * 2048, 0, ""}, true},
        {"one tap, parts, 1568 tiles", {shape(32, 64, 112, 112, 64, 1), geom(2, 0), options(MNN_SCHEME_DIRECT, 0, MNN_GEMM_FP32), parts(64, 64, 1, 3), 0, ""}, false},
    };
    for (const Case& c : cases) {
        const bool ok = in_child([&] {
            fake::takes = [](const std::string&) { return 1.f; };
            mnn_conv_plan_t p = nullptr;
            CHECK(mnn_conv_plan(&c.l.s, &c.l.g, &c.l.o, nullptr, &p) == MNN_OK);
            mnn_conv_plan_destroy(p);
            bool made = false;
            for (size_t b : fake::asked) made |= b == c.l.other_form;
            CHECK(made == c.made);
        });
        std::printf("forms made, %s: %s\n", c.what, ok ? "ok" : "FAILED");
        failures += !ok;
    }
}

}  // namespace

int main()
{
    check_forms_made();
    check_exceptions();
    check_strassen_beside_winograd();
    // F(4,3) 64 -> 96 on 8 x 28 x 28: 392 tiles; U, V and M are kept besides the weights as parts
    const size_t p49 = 8 * 7 * 7, wino = (size_t)36 * 4 * (64 * 96 + 64 * p49 + 96 * p49);
    check_layer("Winograd, fp32", {shape(8, 64, 28, 28, 96, 3), geom(1, 1), options(MNN_SCHEME_WINOGRAD, 4, MNN_GEMM_FP32), 36 * parts(96, 64, 1, 3), wino, "gemm_prepared_kernel"});
    check_layer("Winograd, bf16x3", {shape(8, 64, 28, 28, 96, 3), geom(1, 1), options(MNN_SCHEME_WINOGRAD, 4, MNN_GEMM_BF16X3), 36 * parts(96, 64, 1, 2), wino, "gemm_prepared_kernel"});
    check_layer("pointwise", {shape(8, 128, 28, 28, 256, 1), geom(1, 0), options(MNN_SCHEME_GEMM1X1, 0, MNN_GEMM_FP32), parts(256, 128, 1, 3), (size_t)128 * 256 * 4, "gemm_prepared_kernel"});
    check_layer("sliding window, parts", {shape(1, 100, 14, 14, 100, 3), geom(1, 1), options(MNN_SCHEME_DIRECT, 0, MNN_GEMM_FP32), parts(100, 100, 9, 3), (size_t)900 * 100 * 4, "conv_short_kernelILb1"});
    check_layer("sliding window, fp32 in operand order", {shape(1, 100, 14, 14, 100, 3), geom(1, 1), options(MNN_SCHEME_DIRECT, 0, MNN_GEMM_FP32), (size_t)7 * 4 * 9 * 2048, (size_t)900 * 100 * 4, "conv_short_kernelILb0"});
    check_layer("sliding window, staged patches", {shape(16, 64, 56, 56, 64, 3), geom(1, 1), options(MNN_SCHEME_DIRECT, 0, MNN_GEMM_FP32), parts(64, 64, 9, 3), (size_t)576 * 64 * 4, "conv_patch_kernel"});
    return failures ? 1 : 0;
}
