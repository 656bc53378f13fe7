"""The host side of the library against a stand-in HIP runtime (CPU only):
which device buffers a context holds, when they move, and what a call on a
captured stream does.  host_runtime_stub.cpp says what the stand-in checks."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2403_16125_amd import arena
from paper_2403_16125_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2403_16125_amd", "csrc")
HIP_INCLUDE = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")
OUT = 0x1000        # output arrays: never dereferenced by the stand-in


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "libarena_stub.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-w",
                    "-I", HIP_INCLUDE, "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-Wl,-Bsymbolic", "-o", so,
                    os.path.join(CSRC, "arena_host.cpp"), os.path.join(ROOT, "tests", "host_runtime_stub.cpp")],
                   check=True)
    path, lib = arena._LIB_PATH, arena._lib
    arena._LIB_PATH, arena._lib = so, None
    try:
        s = arena.load()
        s.stub_kappa.restype = ctypes.c_float
        s.stub_live_bytes.restype = ctypes.c_longlong
        yield s
    finally:
        arena._LIB_PATH, arena._lib = path, lib


@pytest.fixture
def ctx(stub):
    stub.stub_capture(0)
    c = arena.arena_create(0)
    yield c
    stub.stub_capture(0)
    arena.arena_destroy(c)


def _bind_jobs(ctx, n_jobs, L):
    arena.arena_bind_jobs(ctx, np.arange(n_jobs + 1) * L, np.full(n_jobs, 64), OUT, OUT, OUT, OUT, OUT)


def _bind(ctx, n_jobs=2, L=40, n_types=8, n_counts=131):
    """2 jobs x 8 types x 131 counts: 256 blocks balanced, 528 under the exact-T rule."""
    _bind_jobs(ctx, n_jobs, L)
    arena.arena_bind_grids(ctx, [1.0] * n_types, [8e10] * n_types, [3e11] * n_types, [2.5e10] * n_types,
                           [8] * n_types, np.arange(n_counts) + 1)
    arena.arena_set_plan_space(ctx, [1, 2, 4], 1e-6)


def _estimate(ctx):
    arena.arena_estimate(ctx, OUT, OUT, OUT)


def _tables(n_types):
    v = np.tile(np.array([0.0, 1e6, 1e9]), (n_types, 2, 1))
    return v, v / 1e11


CHANGES = {
    "rule": lambda c: arena.arena_set_partition_rule(c, arena.PARTITION_EXACT_T),
    "tables": lambda c: arena.arena_set_comm_tables(c, *_tables(8)),
    "cap set": lambda c: arena.arena_set_workspace_limit(c, 1 << 20),
    "cap lifted": lambda c: arena.arena_set_workspace_limit(c, 0),
    "plan space": lambda c: arena.arena_set_plan_space(c, [1, 2, 4, 8], 1e-6),
    "pruning": lambda c: arena.arena_set_bound_pruning(c, False),
}


@pytest.mark.parametrize("cap", [0, 1 << 20])
@pytest.mark.parametrize("change", sorted(CHANGES))
def test_buffers_stay_while_bindings_do(stub, ctx, change, cap):
    """A captured estimate keeps the addresses of the context's buffers, so none of them
    is freed or outgrown by a change of the rule, tables, cap or plan space: after the
    change and an eager estimate the launch recorded first still points at live memory."""
    arena.arena_set_workspace_limit(ctx, cap)
    _bind(ctx)
    _estimate(ctx)
    frees = stub.stub_frees()
    stub.stub_capture(1)
    _estimate(ctx)
    stub.stub_capture(0)
    CHANGES[change](ctx)
    _estimate(ctx)
    arena.arena_set_partition_rule(ctx, arena.PARTITION_BALANCED)
    arena.arena_set_comm_tables(ctx)
    _estimate(ctx)
    assert stub.stub_frees() == frees
    assert stub.stub_faults() == 0


@pytest.mark.parametrize("shape", [(2, 40, 8, 131), (4, 40, 4, 35), (64, 40, 3, 7), (3000, 8, 1, 4), (2, 128, 8, 131)])
def test_split_caches_cover_every_rule(stub, ctx, shape):
    """Without a cap a rule's or the tables' own block count is taken (the caches are
    made for the most any of them needs), and with one the caches stay within it."""
    _bind(ctx, *shape)
    rules = [arena.PARTITION_EXACT_T if shape[1] <= 96 else arena.PARTITION_MEMORY, arena.PARTITION_BALANCED]
    alone = []
    for r in rules:
        c = arena.arena_create(0)
        _bind(c, *shape)
        arena.arena_set_partition_rule(c, r)
        _estimate(c)
        alone.append((stub.stub_blocks(), stub.stub_parts()))
        arena.arena_destroy(c)
    for order in (rules, rules[::-1]):
        for r in order:
            arena.arena_set_partition_rule(ctx, r)
            _estimate(ctx)
            assert (stub.stub_blocks(), stub.stub_parts()) == alone[rules.index(r)]
    assert stub.stub_faults() == 0


def test_caches_stay_within_the_cap(stub, ctx):
    """A cap with room for one block per item and half as much again: accepted, and what
    the context holds afterwards is within it."""
    before = stub.stub_live_bytes()
    limit = 24 * 8448 + (24 << 10)
    arena.arena_set_workspace_limit(ctx, limit)
    _bind(ctx)
    arena.arena_set_partition_rule(ctx, arena.PARTITION_EXACT_T)
    _estimate(ctx)
    pinned = 4 * (3 + 2) + 4 * (16 + 131) + 8 * 8 + 2 * 4 * 8 * 131      # host staging is not counted by the cap
    assert stub.stub_live_bytes() - before - pinned <= limit
    assert stub.stub_blocks() >= 16 and stub.stub_faults() == 0


def _proxy(ctx):
    arena.arena_proxy_estimate(ctx, np.full(8, 2e12), 1e14, 16, OUT, OUT, OUT)


PENDING = {
    "jobs": lambda c: _bind_jobs(c, 50, 40),
    "grids": lambda c: _bind(c, n_counts=200),
    "order": lambda c: arena.arena_set_plan_space(c, [1, 2, 4, 8], 1e-6),
    "tables": lambda c: arena.arena_set_comm_tables(c, *_tables(8)),
    "kappa": lambda c: arena.arena_set_kappa(c, np.full(8 * 131, 1.5, np.float32)),
}


@pytest.mark.parametrize("pending,call", [(p, _estimate) for p in sorted(PENDING)]
                         + [(p, _proxy) for p in ("grids", "jobs", "kappa")])
def test_a_refused_call_releases_nothing(stub, ctx, pending, call):
    """A call that a capture refuses, for whatever is still to be uploaded, has neither
    freed nor made a buffer before it (work recorded earlier in the capture holds
    them) and records nothing."""
    _bind(ctx)
    _estimate(ctx)
    _proxy(ctx)
    PENDING[pending](ctx)
    seen = lambda: (stub.stub_allocs(), stub.stub_frees(), stub.stub_launches(), stub.stub_recorded_copies())
    before = seen()
    stub.stub_capture(1)
    with pytest.raises(arena.ArenaError, match="staging"):
        call(ctx)
    stub.stub_capture(0)
    assert seen() == before
    assert stub.stub_last_dangles() == 0
    call(ctx)
    assert stub.stub_faults() == 0


@pytest.mark.parametrize("call", ["estimate", "proxy"])
def test_pending_factors_are_refused_under_capture(stub, ctx, call):
    """Contention factors that wait for their upload are not recorded into a graph (their
    staging buffer is reused, and nothing would have been copied when the capture ends):
    the call is refused, records nothing, and the next one outside takes the factors."""
    run = dict(estimate=_estimate, proxy=_proxy)[call]
    _bind(ctx)
    run(ctx)
    arena.arena_set_kappa(ctx, np.full(8 * 131, 1.5, np.float32))
    launches, copies = stub.stub_launches(), stub.stub_recorded_copies()
    stub.stub_capture(1)
    with pytest.raises(arena.ArenaError, match="kappa staging"):
        run(ctx)
    stub.stub_capture(0)
    assert stub.stub_launches() == launches and stub.stub_recorded_copies() == copies
    run(ctx)
    assert stub.stub_kappa(0) == 1.5 and stub.stub_kappa(8 * 131 - 1) == 1.5
