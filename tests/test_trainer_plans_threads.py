"""The trainer's plan table under threads: the library's host code of
train_persistent.hip, built with ThreadSanitizer, makes its first plans on eight
threads at once (contexts of their own may do so). No data race is reported and
every thread finds the same shape."""
import glob
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_30497_amd", "csrc")
ROCM = "/opt/rocm"
CLANGXX = os.path.join(ROCM, "llvm", "bin", "clang++")

DRIVER = r"""
#include <pthread.h>
#include <stdint.h>
#include <stdio.h>
#include "mlp_internal.h"
namespace mlp { hipError_t clear_words(const Ctx &, uint64_t *, int64_t) { return hipSuccess; } }
static pthread_barrier_t start;
static int inst[8];
static void *run(void *p) {
    const int i = (int)(intptr_t)p;
    mlp::TrainPlan pl;
    pthread_barrier_wait(&start);
    inst[i] = mlp::plan_train(256, 4096, &pl) ? pl.inst : -1;
    return nullptr;
}
int main() {
    pthread_t t[8];
    pthread_barrier_init(&start, nullptr, 8);
    for (int i = 0; i < 8; ++i) pthread_create(&t[i], nullptr, run, (void *)(intptr_t)i);
    for (int i = 0; i < 8; ++i) pthread_join(t[i], nullptr);
    for (int i = 0; i < 8; ++i) printf("%d ", inst[i]);
    return 0;
}
"""


@pytest.mark.skipif(
    not os.path.exists(CLANGXX) or os.environ.get("MLP_SANITIZED_RUN") == "1" or
    not glob.glob(os.path.join(ROCM, "llvm", "lib", "clang", "*", "lib", "linux", "*tsan*")),
    reason="no ROCm clang or ThreadSanitizer runtime, or inside another sanitizer's run")
def test_first_plans_on_eight_threads(tmp_path):
    (tmp_path / "driver.hip").write_text(DRIVER)
    objs = []
    for src in (os.path.join(CSRC, "train_persistent.hip"), str(tmp_path / "driver.hip")):
        objs.append(str(tmp_path / (os.path.basename(src) + ".o")))
        # host code only: no kernel is built or run here
        subprocess.check_call([os.path.join(ROCM, "bin", "hipcc"), "--offload-arch=gfx950",
                               "--cuda-host-only", "-std=c++17", "-O1", "-g",
                               "-Xarch_host", "-fsanitize=thread",
                               "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
                               "-c", src, "-o", objs[-1]])
    exe = str(tmp_path / "driver")
    # the kernels' code objects are not linked in
    subprocess.check_call([CLANGXX, "-fsanitize=thread"] + objs +
                          ["-L" + os.path.join(ROCM, "lib"), "-lamdhip64", "-lpthread",
                           "-Wl,-rpath," + os.path.join(ROCM, "lib"),
                           "-Wl,--unresolved-symbols=ignore-all", "-o", exe])
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=60)
    assert "ThreadSanitizer" not in r.stdout and r.returncode == 0, r.stdout[-4000:]
    assert r.stdout.split() == ["0"] * 8, r.stdout
