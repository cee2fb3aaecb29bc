"""Host-side checks that need no GPU: the benchmark's one-GPU contract, the
product path failing loudly without its HIP library, and the separation of
the product path from the oracle."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
sys.path.insert(0, ROOT)


def test_bench_refuses_more_than_one_gpu():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in r.stderr


def test_missing_library_fails_loudly(monkeypatch, tmp_path):
    import paper_2305_16317_amd as pd
    monkeypatch.setattr(pd, "_LIB", None)
    monkeypatch.setattr(pd, "lib_path", lambda: str(tmp_path / "absent.so"))
    with pytest.raises(RuntimeError, match="no fallback"):
        pd.load()


def test_product_path_does_not_touch_the_oracle():
    """The package neither imports nor names the oracle (only tests, the
    smoke check and the benchmark's CPU baseline may)."""
    pkg = os.path.join(ROOT, "paper_2305_16317_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hip", ".cpp", ".h")):
                text = open(os.path.join(dirpath, f), encoding="utf-8").read()
                assert "oracle" not in text, os.path.join(dirpath, f)
    code = ("import sys; sys.path.insert(0, %r); import paper_2305_16317_amd, workloads; "
            "print(any(m == 'oracle' or m.startswith('oracle.') for m in sys.modules))" % ROOT)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    assert r.stdout.strip() == "False"


def test_seeded_input_module_holds_no_method_arithmetic():
    """workloads/ (shared by the oracle and the GPU path) only generates
    inputs: it must not name the sampler's quantities."""
    text = open(os.path.join(ROOT, "workloads", "__init__.py"), encoding="utf-8").read()
    for word in ("alphabar", "cumsum", "picard", "drift", "stride"):
        assert word not in text.lower(), word


def test_bench_window_accounting():
    """Window points and history rows of a stride trace (the update's
    algorithmic bytes are priced from them)."""
    import importlib.util
    spec = importlib.util.spec_from_file_location("bench_mod", os.path.join(ROOT, "bench.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    # T = 10, p = 4: windows start at 0, 1, 3, 7 -> sizes 4, 4, 4, 3
    assert b.window_points([1, 2, 4, 3], 4, 10) == 15
    assert b.history_rows([1, 2, 4, 3], 10) == 3
    import workloads as W
    wl = W.WORKLOADS["policy_mlp_dpm15"]
    assert b.update_bytes(wl, 15, False, 3) == 160 * (12 * 15 + 8 * 3)
    assert b.sampler_name(wl).startswith("ParaDPMSolver")
    assert b.metric_name(W.WORKLOADS["latent_ddpm1000_p64"]) == b.METRIC


_PLAN_TEST = r"""
#include <cstdio>
#include <random>
#include <vector>
#include "picard_plan.h"
using namespace pd;
// One loop of T steps whose iterations slide by `strides`: the host's reads fall before or after the
// last queued iteration's stores, or between them (t of one iteration with k of the next, or the
// other way round).  Returns the iterations queued, or a negative number for a wrong end.
static int run(int T, int p, const std::vector<int>& strides, std::mt19937& g) {
    std::vector<int> t(1, 0);
    for (int s : strides) t.push_back(t.back() + s);
    const int last = (int)strides.size();                       // iterations that slide
    auto at = [&](int m) { return m < last ? m : last; };
    int issued = 0, th = 0, kh = 0;
    bool drained = false;
    for (int step = 0; step < 4 * T + 8; ++step) {
        const PicardPlan plan = picard_plan(T, p, issued, th, kh, kh > 0 ? strides[0] : 0, drained);
        if (plan.next == PicardNext::STUCK) return -1;
        if (plan.next == PicardNext::QUEUE) {
            if (plan.n < 1) return -2;
            issued += plan.n;
            drained = false;
            if (issued > T) return -3;
            const int before = at(issued - 1), after = at(issued);
            th = t[g() % 2 ? before : after];
            kh = g() % 2 ? before : after;
        } else {
            if (drained) return -4;
            drained = true;
            th = t[at(issued)];
            kh = at(issued);
        }
        const uint64_t w = pack_progress(th, kh);
        if (progress_t(w) != th || progress_k(w) != kh) return -5;
        if (th >= T) return issued;
    }
    return -6;
}
int main() {
    std::mt19937 g(1);
    for (int i = 0; i < 200000; ++i) {
        const int T = 1 + g() % 20, p = 1 + g() % T, kind = g() % 3;
        std::vector<int> s;
        for (int t = 0; t < T; t += s.back()) {
            const int pe = p < T - t ? p : T - t;
            s.push_back(kind == 0 || s.empty() ? 1 : kind == 1 ? pe : 1 + (int)(g() % pe));
        }
        const int r = run(T, p, s, g);
        if (r < (int)s.size()) {
            std::printf("T %d p %d strides of %zu iterations: %d\n", T, p, s.size(), r);
            return 1;
        }
    }
    return 0;
}
"""


def test_loop_plan_survives_reads_during_the_last_iteration(tmp_path):
    """Whatever mixture of old and new progress the host reads while the last queued iteration
    stores its own, the loop ends with all its iterations run, never as stuck, and never queues
    more than T of them."""
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(_PLAN_TEST)
    inc = os.path.join(ROOT, "paper_2305_16317_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", inc, str(src), "-o", str(exe)], check=True,
                   timeout=300)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
