"""Host code of libcrp.so on the CPU, its HIP calls answered by tests/host/fake_hip.hpp."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    """Compiles tests/host/NAME.cpp against libcrp.so and returns its path."""
    from paper_1307_2643_amd import build as B
    pkg = os.path.dirname(B.LIB)
    out = tmp_path_factory.mktemp("host")

    def make(name):
        exe = out / name
        if not exe.exists():
            subprocess.check_call(
                [B.hipcc(), "--offload-arch=" + B.ARCH, "--offload-host-only", "-x", "hip",
                 "-std=c++17", "-O1", "-rdynamic", "-I", os.path.join(pkg, "..", "include"), "-I",
                 os.path.join(pkg, "csrc"), os.path.join(HERE, "host", name + ".cpp"), "-x", "none",
                 B.LIB, "-Wl,-rpath," + pkg, "-o", str(exe)])
        return str(exe)
    return make


def run(exe, *args):
    r = subprocess.run([exe, *args], capture_output=True, text=True, timeout=120)
    print(r.stdout + r.stderr)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


@pytest.mark.parametrize("kernel", ["k_inject_keys", "8k_inject"])
def test_failed_injection_waits_for_its_upload(driver, kernel):
    run(driver("inject_failure"), kernel)


def test_tuner_trials_are_launched_as_large_batches(driver):
    run(driver("tune"), "trials")


@pytest.mark.parametrize("percent,kept", [(1.5, "128 0"), (-1.5, "128 0"), (5.0, "128 3")])
def test_tuner_takes_fewer_waves_only_beyond_the_noise(driver, percent, kept):
    """Three blocks per compute unit instead of the filled unit: kept when they are faster by
    more than the calibration's noise (3 percent), not within it."""
    assert f"kept {kept}\n" in run(driver("tune"), "keep", str(percent))


@pytest.mark.parametrize("n,layout,lanes", [(1, 7, 1), (1024, 7, 1), (40960, 7, 40), (40961, 0, 41),
                                            (65536, 0, 64), (200000, 0, 64)])
def test_linear_layout_keeps_corner_values_of_large_batches_only(driver, n, layout, lanes):
    """Kept corner values (0) from 41 lanes of a wave on, plain gathers (7) below (256 compute
    units, four waves each)."""
    assert f"layout {layout} lanes {lanes} " in run(driver("linear_rule"), str(n))
