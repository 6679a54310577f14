"""Workspace planning on the CPU: the library's host code over a runtime without a
device (tests/cpu/hip_stub.c).  A call that fits the workspace cap in a context of
its own is never refused for what earlier calls of another size left there."""

import json
import os
import random
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
M = 1 << 20
OK, NOMEM = 0, -3


@pytest.fixture(scope="session")
def stub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.run(["gcc", "-O2", "-Wall", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "cpu", "hip_stub.c")],
                   check=True)
    return so


@pytest.fixture(scope="session")
def run(stub):
    from paper_2011_05755_amd import build
    if not os.path.exists(build.LIB):
        build.build()

    def go(scenario):
        r = subprocess.run([sys.executable, os.path.join(HERE, "stub_driver.py"), build.LIB],
                           input=json.dumps(scenario), capture_output=True, text=True, timeout=100,
                           env=dict(os.environ, LD_PRELOAD=stub))
        assert r.returncode == 0, r.stderr[-2000:]
        return json.loads(r.stdout.strip().splitlines()[-1])
    return go


def refs(L, r, T, K, prec, id=0):
    return ["load", dict(L=L, r=r, T=T, K=K, prec=prec, id=id)]


@pytest.mark.parametrize("L,r,T,K,cap", [(76, 35, 1, 50, 384), (128, 62, 3, 100, 512)])
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_averages_after_alignment(run, L, r, T, K, cap, prec):
    N = 100000
    got = run([dict(cap=cap * M, calls=[refs(L, r, T, K, prec), ["align", dict(N=N)], ["averages", dict(N=N)],
                                        ["align", dict(N=N, cc2=True)], ["averages", dict(N=N)]]),
               dict(cap=cap * M, calls=[["classify", dict(L=L, r=r, T=T, K=K, prec=prec, N=N)]])])
    for g in got:
        assert g["codes"] == [OK] * len(g["codes"]), g["errors"]


def test_no_call_is_refused_for_what_others_left(run):
    rng = random.Random(4)
    sizes = [(64, 28), (76, 35), (96, 46), (128, 62), (24, 9), (160, 64)]
    sequences = []
    for _ in range(250):
        calls = []
        for i in range(rng.randint(2, 4)):
            L, r = rng.choice(sizes)
            calls.append(refs(L, r, rng.choice([0, 1, 2, 3, 5]), rng.choice([2, 5, 20, 100, 400, 3000, 12000]),
                              rng.choice(["fp32", "bf16", "fp16"]), i))
            for _ in range(2):
                kind = rng.choice(["align", "align", "averages"])
                calls.append([kind, dict(id=i, N=int(10 ** rng.uniform(0, 5)), cc2=rng.random() < 0.3)])
        n = sum(c[0] == "load" for c in calls)
        calls.append(["batch", dict(stacks=[[i, int(10 ** rng.uniform(0, 4))] for i in range(n)] * 2)])
        sequences.append(dict(cap=rng.choice([2, 4, 16, 64, 128, 256, 384, 512, 1024]) * M, calls=calls))
    # each call by itself: its reference sets (where they load) and the call
    alone = []
    for s in sequences:
        loads = [c for c in s["calls"] if c[0] == "load"]
        for c in s["calls"]:
            need = loads if c[0] == "batch" else [x for x in loads if x[1]["id"] == c[1]["id"] and c[0] != "load"]
            alone.append(dict(cap=s["cap"], calls=need + [c]))
    got, single = run(sequences), iter(run(alone))
    refused = 0
    for s, g in zip(sequences, got):
        for c, code, err in zip(s["calls"], g["codes"], g["errors"]):
            want = next(single)["codes"][-1]
            assert code == want, (s["cap"] // M, c, err)
            refused += code != OK
    assert refused < sum(len(s["calls"]) for s in sequences) / 2   # (most calls do fit)


@pytest.mark.parametrize("r,K", [(4, 350000), (8, 345000), (64, 131500)])
def test_large_reference_sets_launch_within_the_grid_limit(run, r, K):
    # (no launch may have 2^32 work-items; K as the FP32 operand alone is packed in one launch)
    got = run([dict(cap=1 << 40, calls=[refs(160, r, 0, K, "fp32"), ["align", dict(N=3)]])])[0]
    assert got["codes"] == [OK, OK], got["errors"]
    assert got["most_items"] < 1 << 32


@pytest.mark.parametrize("n", [1, 2])
def test_a_failed_wait_frees_every_buffer_once(run, n):
    # sets of three sizes under one id: the third load frees the first set, after the second wait
    loads = [refs(64, 28, 2, K, "fp32") for K in (5, 6, 7)]
    fine, got = run([dict(cap=M << 10, calls=loads),
                     dict(cap=M << 10, calls=loads[:2] + [["fail_sync", dict(n=n)], loads[2]])])
    assert fine["codes"] == [OK] * 3 and got["codes"] == [OK] * 3 + [-4]
    assert got["bad_frees"] == 0 and got["left"] == fine["left"]
