"""What a forward launches, recorded in place of the launches: no device work.

The library is loaded in a process of its own, behind a recorder that takes the place of the few HIP
calls a forward makes."""
import ctypes
import json
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

RECORDER = r"""
#include <stddef.h>
#include <stdio.h>
#include <string.h>
typedef struct { unsigned x, y, z; } grid_t;
static struct { const void *host; const char *name; } known[512];
static struct { const char *name; unsigned long long groups, threads; } seen[256];
static int n_known, n_seen;
static grid_t grid, block;
void **__hipRegisterFatBinary(void *b) { (void)b; static void *m; return &m; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t n, int c, int g) { (void)m; (void)v; (void)h; (void)d; (void)e; (void)n; (void)c; (void)g; }
void __hipRegisterFunction(void **m, const void *f, char *d, const char *name, unsigned t, void *a, void *b, void *c, void *e, int *w) {
    (void)m; (void)d; (void)t; (void)a; (void)b; (void)c; (void)e; (void)w;
    known[n_known].host = f; known[n_known++].name = name;
}
int __hipPushCallConfiguration(grid_t g, grid_t b, size_t l, void *s) { (void)l; (void)s; grid = g; block = b; return 0; }
int __hipPopCallConfiguration(grid_t *g, grid_t *b, size_t *l, void **s) { *g = grid; *b = block; *l = 0; *s = 0; return 0; }
int hipLaunchKernel(const void *f, grid_t g, grid_t b, void **args, size_t l, void *s) {
    (void)args; (void)l; (void)s;
    const char *name = "?";
    for (int i = 0; i < n_known; ++i) if (known[i].host == f) name = known[i].name;
    if (n_seen < 256) {
        seen[n_seen].name = name;
        seen[n_seen].groups = (unsigned long long)g.x * g.y * g.z;
        seen[n_seen++].threads = (unsigned long long)b.x * b.y * b.z;
    }
    return 0;
}
int hipGetLastError(void) { return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetDevicePropertiesR0600(void *p, int d) { (void)p; (void)d; return 1; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *q) { (void)d; (void)s; (void)n; (void)k; (void)q; return 0; }
int recorded(void) { return n_seen; }
const char *recorded_name(int i) { return seen[i].name; }
unsigned long long recorded_groups(int i) { return seen[i].groups; }
unsigned long long recorded_threads(int i) { return seen[i].threads; }
void recorded_clear(void) { n_seen = 0; }
"""


def record(recorder_path, cases):
    """The launches of each case's forward, [name, workgroups, threads of one]; runs in the child process."""
    import numpy as np
    import torch  # noqa: F401    (its own HIP calls are bound before the recorder comes)
    sys.path.insert(0, os.path.dirname(HERE))
    from paper_2603_28768_amd import binding
    rec = ctypes.CDLL(recorder_path, mode=ctypes.RTLD_GLOBAL)
    rec.recorded_name.restype = ctypes.c_char_p
    rec.recorded_groups.restype = rec.recorded_threads.restype = ctypes.c_uint64
    lib = binding.lib()
    out = []
    for c in cases:
        D, E, k = c.get("D", 1), c["E"], c["k"]
        plan = binding.Plan(np.arange(E, 2 * E, dtype=np.int64)[None, None], D, c.get("replicas", 0))
        assert plan.layer(0)["n_slots"] == E + c.get("replicas", 0)
        a = binding.FwdArgs()
        a.dtype = binding.CRAFT_BF16 if c["dtype"] == "bf16" else binding.CRAFT_F32
        a.T, a.H, a.I, a.k, a.renormalize, a.max_rows = c["T"], c["H"], c["I"], k, 1, c.get("max_rows", 0)
        somewhere = 1 << 40                        # aligned, not null, never read
        a.x = a.out = a.w_gate = a.w_up = a.w_down = a.workspace = a.tables = somewhere
        if c.get("gate"):
            a.w_router = somewhere
        else:
            a.logits = somewhere
        if c.get("packed"):
            a.w_gateup_packed = a.w_down_packed = somewhere
            a.tile_rows_gateup = c.get("tile_rows", 0)
        n = ctypes.c_size_t()
        assert lib.craft_plan_tables_bytes(plan._h, 0, 0, ctypes.byref(n)) == 0
        assert lib.craft_plan_tables_upload(plan._h, 0, 0, ctypes.c_void_p(somewhere), n.value, None) == 0
        assert lib.craft_moe_rank_forward_workspace(plan._h, 0, 0, ctypes.byref(a), ctypes.byref(n)) == 0
        a.workspace_bytes = n.value
        rec.recorded_clear()
        assert lib.craft_moe_rank_forward(plan._h, 0, 0, ctypes.byref(a), None) == 0
        out.append([[rec.recorded_name(i).decode(), rec.recorded_groups(i), rec.recorded_threads(i)]
                    for i in range(rec.recorded())])
    return out


@pytest.fixture(scope="module")
def launches_of(tmp_path_factory):
    where = tmp_path_factory.mktemp("recorder")
    source, so = str(where / "recorder.c"), str(where / "librecorder.so")
    with open(source, "w") as f:
        f.write(RECORDER)
    subprocess.check_call(["gcc", "-O1", "-fPIC", "-shared", source, "-o", so])

    def ask(*cases):
        res = subprocess.run([sys.executable, os.path.abspath(__file__), so, json.dumps(cases)],
                             capture_output=True, text=True, timeout=600)
        assert res.returncode == 0, (res.stdout + res.stderr)[-3000:]
        return json.loads(res.stdout.splitlines()[-1])
    return ask


def test_combine_reaches_every_row_of_a_very_large_batch(launches_of):
    # a launch has fewer than 2^32 threads: of one with more only the remainder would run.  Rows of one and
    # of several pieces on both sides of that, and few rows of very many pieces
    shapes = [("bf16", (1 << 25) - 4, 1024, 1), ("bf16", 1 << 25, 1288, 2), ("f32", 1 << 25, 644, 2), ("bf16", 1 << 24, 4096, 4),
              ("bf16", (1 << 26) + 5, 8, 1), ("bf16", 1024, 1 << 26, 1 << 16), ("bf16", 4096, 7168, 7)]
    found = launches_of(*[dict(dtype=dt, T=T, H=H, I=8, E=2, k=1, D=2, max_rows=64) for dt, T, H, _ in shapes])
    for (dt, T, H, pieces), launches in zip(shapes, found):
        combine = [l for l in launches if "combine" in l[0]]
        assert all(groups * threads < 1 << 32 for _, groups, threads in launches), (dt, T, H, launches)
        assert all(threads == 256 for _, _, threads in combine)
        assert sum(groups for _, groups, _ in combine) == (T + 3) // 4 * pieces, (dt, T, H, combine)


def test_combine_sends_no_wave_for_little(launches_of):
    # pieces of a row, 2 KiB or 3
    shapes = [("bf16", 64, 1024, 1), ("bf16", 64, 1032, 1), ("bf16", 64, 1280, 1), ("bf16", 64, 1288, 2), ("f32", 5000, 640, 1), ("f32", 5000, 644, 2),
              ("bf16", 16384, 2056, 3), ("bf16", 16384, 3072, 3), ("bf16", 16384, 3080, 3), ("bf16", 4095, 3080, 4), ("bf16", 4096, 4088, 3),
              ("bf16", 16384, 4096, 4), ("bf16", 16384, 4104, 3), ("bf16", 16384, 4616, 5), ("bf16", 32768, 7168, 7), ("bf16", 16384, 7176, 5),
              ("f32", 16384, 1540, 3)]
    found = launches_of(*[dict(dtype=dt, T=T, H=H, I=8, E=2, k=1, D=2, max_rows=64) for dt, T, H, _ in shapes])
    for (dt, T, H, pieces), launches in zip(shapes, found):
        assert [l[1] for l in launches if "combine" in l[0]] == [(T + 3) // 4 * pieces], (dt, T, H)


def test_a_gate_of_few_tiles_starts_no_other_workgroups(launches_of):
    # (they go round the XCDs by their number: two tiles padded to eight kept to two of them)
    shapes = [(129, 34, 464, 4), (132, 66, 488, 4), (134, 199, 456, 4), (226, 33, 2016, 64)]
    found = launches_of(*[dict(dtype="bf16", T=T, H=H, I=64, E=E, k=4, D=32, gate=True) for T, E, H, _ in shapes])
    for (T, E, H, groups), launches in zip(shapes, found):
        assert [l[1] for l in launches if "router_logits" in l[0]] == [groups], (T, E, H, launches)


def test_every_gate_shape_takes_the_way_it_stands_for(launches_of):
    from cases import GATE_SHAPES
    from paper_2603_28768_amd import binding
    found = launches_of(*[dict(dtype="bf16", T=T, H=H, I=64, E=E, k=4, D=32, gate=True) for (T, H, E), *_ in GATE_SHAPES])
    for ((T, H, E), (fa, fb), blocks, nparts, nsplit), launches in zip(GATE_SHAPES, found):
        (name, groups, _), = [l for l in launches if "router_" in l[0]]
        assert "router_logits_bf16_kernelILi%dELi%dELb%dE" % (fa, fb, nsplit < nparts) in name, (T, H, E, name)
        units = -(-T // (32 * fb)) * nsplit
        assert groups in (units * blocks, -(-units // 8) * 8 * blocks), (T, H, E, groups)
        n = ctypes.c_size_t()
        assert binding.lib().craft_router_logits_workspace(1, T, H, E, ctypes.byref(n)) == 0 and n.value == nparts * T * E * 4
    assert len({(tile, nsplit < nparts) for _, tile, _, nparts, nsplit in GATE_SHAPES}) == 15     # all there are


def test_the_blocks_of_experts_of_a_gate_in_one_part_meet_only_past_the_cache(launches_of):
    # tiles of 64 tokens x 256 experts in one part: by the grid (tiles x blocks) while 220 MiB hold the
    # activations, padded to eight tiles beyond
    most = (220 << 20) // (2 * 4096)
    shapes = [(most, 384, 4096, (most + 63) // 64 * 2), (most + 1, 384, 4096, ((most + 64) // 64 + 7) // 8 * 8 * 2),
              (16401, 300, 1024, 257 * 2)]
    found = launches_of(*[dict(dtype="bf16", T=T, H=H, I=64, E=E, k=4, D=32, gate=True) for T, E, H, _ in shapes])
    for (T, E, H, groups), launches in zip(shapes, found):
        assert [l[1] for l in launches if "router_logits" in l[0]] == [groups], (T, E, H, launches)


DIRECT, SCAN = ["prefix_kernel", "dispatch_direct_kernel"], ["scan_kernel", "dispatch_kernel"]


INDICES = [
    (1024, 64, 2048, ["dispatch_direct_kernel"]), (1024, 64, 2049, SCAN),      # from the blocks' counts alone
    (1025, 64, 72, DIRECT), (8192, 100, 104, DIRECT), (65536, 40, 48, DIRECT), (65537, 40, 48, SCAN),
    (65536, 64, 2048, DIRECT), (65536, 64, 2049, SCAN),
    # one group of experts and more than three passes over the slots: scanned by a single workgroup
    (1025, 64, 1537, SCAN), (8192, 64, 2048, SCAN), (4096, 33, 2048, SCAN),
    (8192, 64, 1536, DIRECT), (8193, 64, 1537, DIRECT), (4096, 65, 2048, DIRECT)]


def test_which_launches_make_the_dispatch_indices(launches_of):
    found = launches_of(*[dict(dtype="f32", T=T, H=64, I=32, E=E, k=2, D=64, replicas=slots - E) for T, E, slots, _ in INDICES])
    for (T, E, slots, indices), launches in zip(INDICES, found):
        names = [l[0] for l in launches if any(w in l[0] for w in ("prefix", "scan", "dispatch"))]
        assert len(names) == len(indices) and all(i in n for i, n in zip(indices, names)), (T, E, slots, names)


# dtype, tokens, experts, gate, the caller's own tile heights -> instance of the routing dispatch: rows
# copied, 64-expert groups up to, parts added; None: routed by a launch of its own
ROUTED = [
    ("bf16", 1, 8, False, False, (1, 1, 0)), ("bf16", 32, 64, True, False, (1, 1, 1)), ("bf16", 32, 65, False, True, (0, 2, 0)),
    ("bf16", 32, 128, True, True, (0, 2, 1)), ("bf16", 8, 129, True, False, (1, 4, 1)), ("bf16", 32, 256, False, False, (1, 4, 0)),
    ("bf16", 32, 257, True, True, (0, 6, 1)), ("bf16", 32, 384, True, False, (1, 6, 1)), ("f32", 32, 384, False, False, (0, 6, 0)),
    ("f32", 32, 64, True, False, (0, 1, 0)),               # a gate that is not split
    ("bf16", 33, 64, True, False, None), ("bf16", 32, 385, False, False, None), ("bf16", 32, 512, True, False, None)]


def test_which_batches_are_routed_by_the_dispatch(launches_of):
    found = launches_of(*[dict(dtype=dt, T=T, H=2048, I=64, E=E, k=4, D=min(E, 32), gate=gate, packed=dt == "bf16",
                               tile_rows=128 if tiled else 0) for dt, T, E, gate, tiled, _ in ROUTED])
    for (dt, T, E, gate, tiled, instance), launches in zip(ROUTED, found):
        names = [l[0] for l in launches]
        routed = [n for n in names if "12route_kernel" in n]
        dispatch, = [n for n in names if "dispatch_direct_kernel" in n]
        assert len(routed) == (instance is None), names
        if instance is not None:
            assert "Lb%dELi%dELb%dE" % instance in dispatch, (dt, T, E, gate, tiled, dispatch)
        else:
            assert "Li0E" in dispatch


def test_a_batch_of_more_than_2048_slots_is_routed_by_a_launch_of_its_own(launches_of):
    many, few = launches_of(*[dict(dtype="f32", T=32, H=64, I=32, E=64, k=4, D=64, replicas=r) for r in (1985, 1984)])
    assert any("12route_kernel" in l[0] for l in many) and not any("12route_kernel" in l[0] for l in few)


if __name__ == "__main__":
    print(json.dumps(record(sys.argv[1], json.loads(sys.argv[2]))))
