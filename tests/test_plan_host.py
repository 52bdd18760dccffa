"""The host side of plans and of the allocation-free call, on the CPU:
mivit_api.cpp and mivit_noalloc.hip built for the host alone, over a stand-in HIP runtime and stand-in launchers (tests/host/plan_driver.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc")
CLANG = "/opt/rocm/lib/llvm/bin/clang++"
pytestmark = pytest.mark.skipif(HIPCC is None or not os.path.exists(CLANG),
                                reason="ROCm compilers not available")


@pytest.fixture(scope="module")
def out(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("plan_host")
    objs, procs = [], []
    for s in ("paper_2011_13579_amd/csrc/mivit_api.cpp",
              "paper_2011_13579_amd/csrc/mivit_noalloc.hip", "tests/host/plan_driver.cpp"):
        name = os.path.splitext(os.path.basename(s))[0]
        objs.append(str(tmp / (name + ".o")))
        # the one with a kernel: its (absent) device code under a fixed symbol
        cuid = ["-fuse-cuid=none"] if s.endswith(".hip") else []
        procs.append(subprocess.Popen(
            [HIPCC, "-x", "hip", "--offload-host-only"] + cuid + ["-O1", "-std=c++17", "-c",
             os.path.join(ROOT, s), "-o", objs[-1]], stderr=subprocess.PIPE, text=True))
    for p in procs:
        _, err = p.communicate(timeout=600)
        assert p.returncode == 0, err[-4000:]
    exe = str(tmp / "plan_driver")
    subprocess.run([CLANG] + objs + ["-o", exe], check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    values = dict(ln.split(" ", 1) for ln in r.stdout.splitlines())
    assert values["done"] == "1"
    return values


@pytest.mark.parametrize("name,frames,parts", [
    ("k7_split", 64, 7), ("k7_open", 256, 8), ("k7_float", 512, 1), ("k9_split", 512, 8),
    ("k9_rate_quarter", 512, 8)])
def test_plan_creation_copies_tables_only(out, name, frames, parts):
    """A plan costs a call that builds one (the first decode of a shape, the
    first push of a stream) its allocations and copies: one allocation per part
    beside the plan's two, and no more bytes than the tables that the host
    writes: per item 64 bytes and its 40 of gradient facts, per wavefront entry
    a unit of 32 for each of up to `parts` parts and the entry itself, and 16
    for the traceback."""
    assert out["tables.%s.status" % name] == "0"
    assert int(out["tables.%s.allocations" % name]) <= 3
    assert int(out["tables.%s.copied" % name]) <= 1024 + 512 * 104 + frames * (32 * (parts + 1) + 32)
    assert out["tables.%s.left" % name] == "0"


@pytest.mark.parametrize("code", ["k7", "k5"])
def test_open_radix_falls_back_to_what_fits(out, code):
    """Frames of different lengths take twice the survivors in packed radix 4:
    where that does not fit, a plan that leaves the radix open runs radix 2."""
    assert out["open_radix_memory." + code] == "0 rot"
    assert out["open_radix_memory.%s.left" % code] == "0"


@pytest.mark.parametrize("name", ["k9_f32.wide1", "k9_f32.wide2", "k9_f32.wide4", "k9_f32.generic2",
                                  "k8_f32.wide1", "k8_f32.wide2", "k8_f32.generic2",
                                  "k9_f16.wide1", "k9_f16.wide4", "k8_f16.wide1", "k8_f16.wide2"])
def test_tuner_tries_every_form_of_the_float_kernel(out, name):
    """K = 8, 9 float frames run over one, two or four wavefronts each: the
    tuner keeps whichever is fastest, also one per frame where the batch alone
    would be spread over four."""
    assert out["tuned." + name] == "0 " + name.split(".")[1]


@pytest.mark.parametrize("name,runs,text", [
    ("k9_few", "wide4", "4 wavefronts per item (automatic: one wavefront per item on a "
     "full device), 4 items, 16 wavefronts"),
    ("k9_many", "wide1", "one wavefront per item, 4096 items, 4096 wavefronts"),
    ("k9_v6", "wide2", "two wavefronts per item, 4 items, 8 wavefronts"),
    ("k9_v7", "wide4", "four wavefronts per item, 4 items, 16 wavefronts"),
    ("k8_few", "wide2", "2 wavefronts per item (automatic: one wavefront per item on a "
     "full device), 4 items, 8 wavefronts"),
    ("k8_f16", "wide1", "one wavefront per item, 4096 items, 4096 wavefronts")])
def test_description_names_what_runs(out, name, runs, text):
    assert out["described." + name].startswith(runs + ": ")
    assert out["described." + name].endswith(text)


@pytest.mark.parametrize("name", ["k3_f32", "k4_i8", "k5_i8", "k7_i8", "k7_f16", "k8_i8", "k9_f32",
                                  "k9r4_i8"])
def test_allocation_free_call_takes_what_its_limit_allows(out, name):
    """The largest batch whose items, entries, pairs, end states and survivors
    fit 64 MiB is decoded and one frame more is refused: tables that the
    traceback adds do not count, and end within the array."""
    assert out["noalloc_limit." + name] == "0 0"
    assert int(out["noalloc_room." + name]) <= 70 << 20


@pytest.mark.parametrize("name,kernel", [
    ("k7_short", "rot"), ("k7_long", "r4p"), ("k7_few", "rot"), ("k7_many", "r4p"),
    ("k5_long", "r4p"), ("k5_many", "r4p"), ("k9_i8", "wpk1"), ("k9_f32", "wide4"),
    ("k8_f32_many", "wide1")])
def test_allocation_free_call_runs_the_plans_kernel(out, name, kernel):
    assert out["same_kernel." + name] == "00 %s %s" % (kernel, kernel)
