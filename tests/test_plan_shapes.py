"""Plans over random shapes, on the CPU.

The streaming verify is planned only where the device holds two workgroups of
it per CU, which a host without a GPU cannot ask.  The host code is therefore
built once more with an MI355X's occupancies in place of the queries (one
workgroup per CU of the fused kernels, two of the streaming one), linked to the
library's kernels, which no test here launches."""
import os
import random
import shutil
import subprocess

import pytest

from paper_2607_27735_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2607_27735_amd")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
OCCUPANCY = {"stream_blocks_per_cu": ("", 2), "fused_blocks_per_cu": ("int", 1), "select_blocks_per_cu": ("int", 1)}


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not shutil.which("g++") or not os.path.exists(B.LIB_PATH):
        pytest.skip("g++ or the built library not available")
    d = tmp_path_factory.mktemp("plans")
    stub = d / "occupancy.cpp"
    stub.write_text("namespace ssl {\n" + "".join(
        f"int mi355x_{f}({arg}) {{ return {n}; }}\n" for f, (arg, n) in OCCUPANCY.items()) + "}\n")
    out = str(d / "libplans.so")
    csrc = os.path.join(PKG, "csrc")
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include",
                    "-I", os.path.join(ROOT, "include"), "-I", csrc, *[f"-D{f}=mi355x_{f}" for f in OCCUPANCY],
                    os.path.join(csrc, "api.cpp"), os.path.join(csrc, "controller.cpp"), str(stub), "-Wl,-Bsymbolic",
                    B.LIB_PATH, f"-Wl,-rpath,{PKG}", f"-L{ROCM}/lib", "-lamdhip64", f"-Wl,-rpath,{ROCM}/lib",
                    "-o", out], check=True)
    saved = B._lib
    yield B.load(out)
    B._lib = saved


def plan(lib, hq, hkv, ctx, ql, mode=B.VERIFY_AUTO, cus=0, per_head=False):
    """(schedule, chunk, items, workspace bytes) or the status."""
    B._lib = lib
    B.set_cu_budget(cus)
    shape = B.Shape(len(ctx), hq, hkv, 128, max(ctx), max(ql))
    p = B.make_params(0.088, budget=64, verify_mode=mode, per_head=per_head)
    try:
        return B.verify_plan(shape, p, ctx, ql) + (B.verify_workspace_bytes(shape, p, ctx, ql),)
    except B.SSLError as e:
        return e.status
    finally:
        B.set_cu_budget(0)


def shapes(seed, n):
    rng = random.Random(seed)
    for _ in range(n):
        hkv, g = rng.choice([1, 2, 4, 8, 16]), rng.choice([1, 1, 2, 3, 4, 4, 5, 8, 8, 16, 31, 40, 64])
        hi = int(10 ** rng.uniform(0, 5.6))
        lo = max(1, hi // rng.choice([1, 2, 20]))
        ctx = [rng.randint(lo, hi) for _ in range(rng.choice([1, 1, 2, 3, 4, 8, 16, 40]))]
        q_hi = rng.choice([1, 2, 5, 8, 12, 16, 33, 64])
        yield hkv * g, hkv, ctx, [min(t, rng.randint(1, q_hi)) for t in ctx], rng.choice([0, 0, 0, 1, 2, 8, 24, 100])


def test_every_shape_has_a_plan(lib):
    """AUTO and TWO_SWEEP take every shape within the limits, whatever the CU
    budget (17 row blocks under a budget of 8 CUs among them), and every
    schedule is met."""
    # (hq, hkv, ctx, q_len, CU budget)
    fixed = [(62, 2, [188], [17], 8), (31, 1, [188], [17], 8), (64, 8, [20011], [16], 0)]
    met = set()
    for hq, hkv, ctx, ql, cus in fixed + list(shapes(1, 4000)):
        for mode in (B.VERIFY_AUTO, B.VERIFY_TWO_SWEEP):
            r = plan(lib, hq, hkv, ctx, ql, mode, cus)
            assert not isinstance(r, int), (hq, hkv, ctx, ql, cus, r)
            sch, chunk, items, nbytes = r
            assert mode == B.VERIFY_AUTO or sch == B.VERIFY_TWO_SWEEP
            assert chunk >= 32 and items >= len(ctx) * hkv and nbytes > 0
            met.add(sch)
    assert met == {B.VERIFY_ONE_SWEEP, B.VERIFY_TWO_SWEEP, B.VERIFY_ONE_SWEEP_PERSISTENT}


# (hq, hkv, contexts, positions, per head, schedule): measured on an MI355X, the form that is faster
@pytest.mark.parametrize("hq,hkv,ctx,q_len,per_head,schedule", [
    (64, 8, [20011], 16, False, B.VERIFY_ONE_SWEEP_PERSISTENT), (64, 8, [9246] * 3, 7, True, B.VERIFY_TWO_SWEEP),
    (32, 8, [42384] * 2, 12, False, B.VERIFY_TWO_SWEEP), (32, 8, [9000] * 4, 12, False, B.VERIFY_ONE_SWEEP_PERSISTENT),
    (64, 8, [32768] * 4, 16, False, B.VERIFY_TWO_SWEEP), (32, 8, [131072], 9, False, B.VERIFY_TWO_SWEEP),
    (32, 8, [70000], 7, False, B.VERIFY_ONE_SWEEP_PERSISTENT)])
def test_streaming_or_two_sweeps(lib, hq, hkv, ctx, q_len, per_head, schedule):
    r = plan(lib, hq, hkv, ctx, [q_len] * len(ctx), per_head=per_head)
    assert r[0] == schedule, r
