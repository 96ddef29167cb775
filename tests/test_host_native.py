"""Host-side native checks, built with AddressSanitizer and UBSan (CPU only).

* The C ABI layer (``csrc/api.cpp``) linked with host stand-ins for the HIP
  runtime and the kernel launchers (``tests/native/abi_stubs.cpp``): every
  entry point runs through validation to its dispatch, and the resolved
  problem is checked (``tests/native/abi_driver.cpp``).
* The persistent block-indexer work split (``csrc/persistent_units.hpp``)
  replayed over many sequence lengths, first groups and grid sizes: every
  (query group, key tile) unit is covered exactly once.
* The kernels that look for NaN in their results: the device code of the build's
  own flags holds no assumption that a value is not NaN.
* The oracle's C source built with both sanitizers and run under the oracle
  pin tests.
"""
import os
import subprocess
import sys

import pytest

from paper_2606_07703_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_07703_amd", "csrc")
NATIVE = os.path.join(ROOT, "tests", "native")
SAN = ["-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-fno-omit-frame-pointer"]
HIP_HOST = ["-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include"]


def _gxx(out, srcs, extra=()):
    cmd = ["g++", "-std=c++17", "-O1", "-g", *SAN, *HIP_HOST, "-I", os.path.join(ROOT, "include"),
           "-I", CSRC, *srcs, "-o", out, *extra]
    subprocess.run(cmd, check=True, capture_output=True, text=True)


def _run(exe, env=None):
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


def test_abi_layer_under_sanitizers(tmp_path):
    exe = str(tmp_path / "abi_driver")
    _gxx(exe, [os.path.join(CSRC, "api.cpp"), os.path.join(NATIVE, "abi_stubs.cpp"),
               os.path.join(NATIVE, "abi_driver.cpp")])
    assert "abi ok" in _run(exe)


def test_persistent_split_covers_every_unit_once(tmp_path):
    exe = str(tmp_path / "unit_cover")
    _gxx(exe, [os.path.join(NATIVE, "unit_cover.cpp")])
    assert "cover ok" in _run(exe)


def test_mass_grid_holds_every_item_once(tmp_path):
    exe = str(tmp_path / "mass_grid_cover")
    _gxx(exe, [os.path.join(NATIVE, "mass_grid_cover.cpp")])
    assert "grid ok" in _run(exe)


def _rule(tmp_path, name, problems):
    """What the rule program `name` prints for each of the problems."""
    exe = str(tmp_path / name)
    _gxx(exe, [os.path.join(NATIVE, name + ".cpp")])
    text = "\n".join(" ".join(map(str, s)) for s in problems)
    r = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    out = [tuple(map(int, ln.split())) for ln in r.stdout.splitlines()]
    assert len(out) == len(problems)
    return out


def test_topk_threads_where_fewer_are_slower(tmp_path):
    """S, q_offset, block_q, k, window -> threads: problems measured slower with
    fewer threads (many positions to write, few rows with any to choose), and the
    ones fewer threads are for."""
    want = {(4096, 0, 1, 4080, 0): 512, (4096, 2560, 1, 4080, 0): 512,
            (2048, 0, 1, 2032, 0): 512, (8192, 7680, 1, 2048, 0): 512,
            (16384, 15872, 1, 2048, 0): 512, (16384, 15872, 1, 64, 128): 512,
            (8192, 4096, 1, 6144, 0): 256, (4096, 0, 1, 3072, 0): 256,
            (2048, 0, 1, 64, 0): 128, (4096, 0, 1, 2560, 0): 128, (8192, 0, 1, 2048, 0): 128,
            (4096, 0, 1, 512, 0): 64, (16384, 0, 1, 2048, 0): 256,
            (32768, 0, 64, 2048, 128): 512, (100, 0, 64, 2_000_000_000, 0): 512}
    got = _rule(tmp_path, "topk_rule", list(want))
    assert [g for g, in got] == list(want.values()), list(zip(want.items(), got))


def test_masked_shapes_take_the_masked_kernel(tmp_path):
    """The shapes of the masked kernel's GPU tests are on its side of the rule, in
    both of its forms, and calls it was measured slower at are not."""
    from test_gpu_next import MASKED
    taken = [s[:2] + s[3:7] for s in MASKED] + [(3000, 0, 64, 16, 128, 1024)]
    got = _rule(tmp_path, "mask_rule", taken)
    assert all(m for m, _ in got), list(zip(taken, got))
    assert {(s[4], split) for s, (_, split) in zip(taken, got)} == {
        (64, 0), (64, 1), (128, 0), (128, 1), (256, 0)}
    # 1024 queries at one head a group: 299 us against 219 gathered; rows of 64
    # entries; a support row too long to count in 32 bits
    gathered = [(4096, 3072, 8, 8, 128, 1024), (4096, 3072, 8, 8, 128, 2048),
                (2048, 0, 32, 8, 128, 64), (64, 0, 1, 1, 64, 2_000_000_000)]
    assert not any(m for m, _ in _rule(tmp_path, "mask_rule", gathered))


@pytest.mark.parametrize("name", ["dense_chunk_mfma.hip", "sparse_mask_mfma.hip"])
def test_kernels_that_look_for_nan_honour_it(tmp_path, name):
    out = str(tmp_path / "dev.ll")
    r = subprocess.run([build.HIPCC, *build.CFLAGS, *build.FILE_FLAGS.get(name, []),
                        "--cuda-device-only", "-S", "-emit-llvm", "-Xclang", "-disable-llvm-passes",
                        os.path.join(CSRC, name), "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    with open(out) as f:
        text = f.read()
    assert "amdgpu_kernel" in text
    for assumed in (" nnan", "nofpclass(nan", '"no-nans-fp-math"="true"'):
        assert assumed not in text, assumed


def _runtime(name):
    return subprocess.run(["gcc", f"-print-file-name={name}"], capture_output=True,
                          text=True, check=True).stdout.strip()


def test_oracle_pins_under_sanitizers(tmp_path):
    lib = str(tmp_path / "libsp_oracle_san.so")
    subprocess.run(["gcc", "-O1", "-g", "-std=c99", "-fopenmp", "-fPIC", "-shared", *SAN,
                    os.path.join(ROOT, "oracle", "sp_oracle.c"), "-o", lib, "-lm"],
                   check=True, capture_output=True, text=True)
    asan, ubsan = _runtime("libasan.so"), _runtime("libubsan.so")
    if not (os.path.isabs(asan) and os.path.isabs(ubsan)):
        pytest.skip("sanitizer runtimes not found")
    env = dict(os.environ, SP_ORACLE_LIB=lib, LD_PRELOAD=f"{asan}:{ubsan}",
               ASAN_OPTIONS="detect_leaks=0", UBSAN_OPTIONS="halt_on_error=1:print_stacktrace=1")
    probe = ("import oracle; oracle._load(); import sys; "
             "sys.exit(0 if oracle._lib._name == sys.argv[1] else 3)")
    subprocess.run([sys.executable, "-c", probe, lib], check=True, env=env, cwd=ROOT,
                   timeout=120)
    r = subprocess.run([sys.executable, "-m", "pytest", "-x", "-q", "-p", "no:cacheprovider",
                        "tests/test_oracle_pins.py", "tests/test_oracle_next_pins.py"],
                       capture_output=True, text=True, env=env, cwd=ROOT, timeout=600)
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-3000:]
    assert "passed" in r.stdout
