"""What a pool allocates, where it waits and which kernel it picks: the host side against a HIP runtime that runs on the host
(tests/native/host_pool.cpp), and the same promise - a call is enqueued and returns - on the GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def host_pool(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("no g++ or no HIP headers")
    csrc = os.path.join(ROOT, "paper_2401_06761_amd", "csrc")
    exe = str(tmp_path_factory.mktemp("native") / "host_pool")
    built = subprocess.run([cxx, "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
                            "-I" + csrc, os.path.join(ROOT, "tests", "native", "host_pool.cpp")] +
                           [os.path.join(csrc, f) for f in ("plan.cpp", "apar_pool.cpp", "controller.cpp")] + ["-o", exe], capture_output=True, text=True)
    assert built.returncode == 0, built.stderr[-3000:]
    return exe


@pytest.mark.parametrize("check", ["staging", "creation", "fixed", "prefill", "slices", "partials"])
def test_host_side(host_pool, check):
    ran = subprocess.run([host_pool, check], capture_output=True, text=True, timeout=120)
    assert ran.returncode == 0 and ran.stdout == f"ok: {check}\n", ran.stdout + ran.stderr


def test_the_host_side_names_every_launcher_it_needs(tmp_path):
    """A library built without a kernel's file must not link: no launcher is a symbol that may stay undefined."""
    cxx, nm = shutil.which("g++"), shutil.which("nm")
    if cxx is None or nm is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("no g++, no nm or no HIP headers")
    csrc, obj = os.path.join(ROOT, "paper_2401_06761_amd", "csrc"), str(tmp_path / "apar_pool.o")
    subprocess.run([cxx, "-std=c++17", "-c", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"), "-I" + csrc,
                    os.path.join(csrc, "apar_pool.cpp"), "-o", obj], check=True, capture_output=True)
    launchers = [l.split() for l in subprocess.run([nm, "-C", obj], check=True, capture_output=True, text=True).stdout.splitlines() if "apar::launch_" in l]
    assert len(launchers) >= 6 and all(kind == "U" for kind, *_ in launchers), launchers


@pytest.mark.gpu
def test_first_staged_calls_return_before_the_work_they_wait_behind():
    """A new pool's first four staged calls (there are four staging slots), on a stream with work ahead of them, are
    enqueued and return: none waits for that work."""
    import torch

    import paper_2401_06761_amd as ap

    def calls(pool, live, q, k):
        out, v = torch.empty_like(q), torch.empty_like(k)
        for _ in range(2):
            ap.apar_decode_attention(pool.handle, q, live, out)
            ap.apar_read_kv_rows(pool.handle, live[0], 0, 100, k, v)

    def pool_of_threads():
        pool = ap.Pool(8, 8, 128, "bf16", 1400)
        live = []
        for i in range(120):
            live.append(ap.apar_thread_create(pool.handle))
            ap.apar_append_kv(pool.handle, live[-1], rows[:100 + i % 50], rows[:100 + i % 50])
        return pool, live

    rows = torch.randn(150, 8, 128, device="cuda:0").bfloat16()
    q = torch.randn(120, 8, 128, device="cuda:0").bfloat16()
    a = torch.randn(8192, 8192, device="cuda:0").bfloat16()
    b = torch.empty_like(a)
    torch.mm(a, a, out=b)
    with pool_of_threads()[0]:
        pass
    pool, live = pool_of_threads()
    with pool:  # the kernels are loaded by now
        calls(pool, live, q, rows[:100].clone())
        torch.cuda.synchronize()
    pool, live = pool_of_threads()
    with pool:
        k = rows[:100].clone()
        torch.cuda.synchronize()
        for _ in range(100):  # some 90 ms
            torch.mm(a, a, out=b)
        ahead = torch.cuda.Event()
        ahead.record()
        calls(pool, live, q, k)
        assert not ahead.query()
        with ap.Pool(8, 8, 128, "bf16", 1400) as another:  # (nor does creating one; destroying one does)
            assert another.handle and not ahead.query()
        torch.cuda.synchronize()
