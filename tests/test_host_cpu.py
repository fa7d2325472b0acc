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


def test_tuner_tries_what_makes_a_difference_to_the_batch(driver):
    """A batch that is spread over the waves is one launch for all refill thresholds and numbers
    of blocks, which are not tried then; a large one is tried in full waves."""
    def trials(n):
        out = run(driver("tune"), "shapes", str(n)).splitlines()
        return [t.split()[1:] for t in out if t.startswith("trial")], out[-1]
    few, kept = trials(3000)
    assert len(few) == 8 and len(set(map(tuple, few))) == 4      # two of each
    assert {t[5] for t in few} == {"3"} and {t[7] for t in few} == {"4"}
    assert kept.endswith("blocks 0 refill 4")
    many, _ = trials(70000)
    assert {t[5] for t in many} == {"64"} and {t[7] for t in many} == {"1", "4", "16", "64"}


@pytest.mark.parametrize("three,sixteen,kept", [(1.5, 0, "128 blocks 0 refill 4"),
                                                (0, 1.5, "128 blocks 0 refill 4"),
                                                (5, 0, "128 blocks 3 refill 4"),
                                                (0, 5, "128 blocks 0 refill 16")])
def test_tuner_leaves_the_default_only_beyond_the_noise(driver, three, sixteen, kept):
    """Three blocks per compute unit instead of the filled unit, or another refill threshold: kept
    when faster by more than the calibration's noise (3 percent), not within it."""
    assert f"kept block {kept}\n" in run(driver("tune"), "keep", str(three), str(sixteen))


def test_tuner_cache_tells_small_batches_from_large(driver, tmp_path):
    run(driver("tune"), "cache", str(tmp_path / "tune.txt"))


@pytest.mark.parametrize("n,layout,lanes", [(1, 7, 1), (1024, 7, 1), (40960, 7, 40), (40961, 0, 41),
                                            (65536, 0, 64), (200000, 0, 64)])
def test_linear_layout_keeps_corner_values_of_large_batches_only(driver, n, layout, lanes):
    """Kept corner values (0) from 41 lanes of a wave on, plain gathers (7) below (256 compute
    units, four waves each)."""
    assert f"layout {layout} lanes {lanes} " in run(driver("linear_rule"), str(n))
