"""The library's launches against a HIP runtime of the test's own (fake_hip.h): what the
host side does when the current device changes and when a launch fails, without a
GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB_DIR = os.path.join(ROOT, "paper_2603_16536_amd")


def run(tmp_path, program):
    if not os.path.exists(os.path.join(LIB_DIR, "libkamx.so")):
        import __graft_entry__
        __graft_entry__.build()
    src, exe = tmp_path / "launches.cpp", tmp_path / "launches"
    src.write_text(program)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.dirname(os.path.abspath(__file__)), str(src), "-o", str(exe),
                    os.path.join(LIB_DIR, "libkamx.so"), f"-Wl,-rpath,{LIB_DIR}", "-rdynamic"], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    print(out.stdout + out.stderr)
    assert out.returncode == 0
    return out.stdout


DEVICES = r"""
#include "fake_hip.h"
#include "kamx.h"
#define CHECK(x) do { if ((x) != KAMX_OK) { std::printf("%s: %s\n", #x, kamx_last_error()); return 1; } } while (0)
// one world of a free body that takes contacts, and one with a loop of joints
static int use(int contacts, int solver) {
    kamx_body_desc b[2] = {{0, 1.f, {1.f, 1.f, 1.f}}, {0, 1.f, {1.f, 1.f, 1.f}}};
    kamx_joint_desc j{};
    j.body_b = 1;
    j.frame_a[6] = j.frame_b[6] = 1.f;
    j.limit_lo = j.limit_hi = __builtin_nanf("");
    kamx_params p;
    kamx_default_params(&p);
    p.linear_solver = solver;
    kamx_model m;
    CHECK(kamx_model_create(b, 2, &j, 1, nullptr, 0, nullptr, 1, contacts, &p, &m));
    CHECK(kamx_step(m, 1, nullptr));
    CHECK(kamx_step(m, 3, nullptr));
    float target = 0.f;
    CHECK(kamx_forward_kinematics(m, &target, 5, 1e-6f, nullptr, nullptr, nullptr));
    CHECK(kamx_model_destroy(m));
    return 0;
}
int main() {
    for (int round = 0; round < 2; ++round)
        for (fake::device = 0; fake::device < 3; ++fake::device) {
            for (int contacts : {4, 30, 40, 50, 64})
                for (int solver : {KAMX_SOLVER_DENSE, KAMX_SOLVER_SPARSE})
                    if (use(contacts, solver)) return 1;
            // a network whose rows of 32 take more than 64 KB
            kamx_mlp n;
            std::vector<float> x(5000 * 1300), y(5000 * 20);
            CHECK(kamx_mlp_create(1300, 256, 20, 5000, 1, &n));
            CHECK(kamx_mlp_forward(n, x.data(), 5000, y.data(), nullptr));
            CHECK(kamx_mlp_train_step(n, x.data(), y.data(), 5000, 1e-3f, nullptr, nullptr));
            CHECK(kamx_mlp_destroy(n));
        }
    size_t large = 0;
    for (const fake::Launch &l : fake::launches) large += l.lds > 65536;
    std::printf("%zu launches, %zu with more than 64 KB of LDS\n", fake::launches.size(), large);
    return fake::refused != 0 || large < 6 * 25;
}
"""


def test_large_lds_on_every_device(tmp_path):
    """A kernel with more than 64 KB of LDS is launched only where the limit has been
    raised for it on the device that is current, also when another device used it
    first."""
    run(tmp_path, DEVICES)


ADAM = r"""
#include <cmath>
#include "fake_hip.h"
#include "kamx.h"
static int count, fail_at = -1;
static float c1, c2;
static const float kLr = 0.12345f;
// the bias corrections of the update: beside the learning rate in the arguments
static void seen(const fake::Launch &l) {
    if (l.name.find("adam_kernel") != std::string::npos) {
        c1 = *(float *)l.args[6];
        c2 = *(float *)l.args[7];
    } else if (l.name.find("grads_kernel") != std::string::npos) {
        float v[48];
        std::memcpy(v, l.args[0], sizeof(v));
        for (int k = 0; k + 2 < 48; ++k)
            if (v[k] == kLr) {
                c1 = v[k + 1];
                c2 = v[k + 2];
            }
    }
}
static bool failing(const std::string &) { return count++ == fail_at; }
int main() {
    fake::on_launch = seen;
    fake::fail_launch = failing;
    for (int hidden : {64, 576}) {
        kamx_mlp n;
        std::vector<float> x(64 * 10), y(64 * 10);
        float loss;
        if (kamx_mlp_create(10, hidden, 10, 64, 1, &n) != KAMX_OK) return 1;
        int good = 0, failed = 0;
        for (int k = 0; k < 40; ++k) {
            // every launch of a step fails in one of the odd calls
            fail_at = k % 2 ? k / 2 : -1;
            count = 0;
            c1 = c2 = 0.f;
            const bool ok = kamx_mlp_train_step(n, x.data(), y.data(), 64, kLr, &loss, nullptr) == KAMX_OK;
            if (!ok) {
                ++failed;
                continue;
            }
            ++good;
            const float w1 = (float)(1.0 - std::pow(0.9, good)), w2 = (float)(1.0 - std::pow(0.999, good));
            if (c1 != w1 || c2 != w2) {
                std::printf("%d hidden, %d updates, %d failed: corrections %g %g, not %g %g\n", hidden, good, failed, c1, c2, w1, w2);
                return 1;
            }
        }
        std::printf("%d hidden: %d updates, %d failed\n", hidden, good, failed);
        if (failed < 2) return 1;
    }
    return 0;
}
"""


def test_failed_training_steps_do_not_count(tmp_path):
    """Adam's bias corrections count the updates that were launched."""
    run(tmp_path, ADAM)
