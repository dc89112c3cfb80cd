"""GPU parity: the HIP path, called through the C ABI, against the CPU checker on the same
seeded inputs.  Integer results (ids, counts, dispatch indices) are compared bit for bit;
gate weights to 1e-5 relative; the layer output to max|gpu-ref| <= tol * max|ref| with
tol = 1e-2 for bf16 storage (fp32 accumulation) and 1e-4 for fp32 storage."""

import numpy as np
import pytest

import oracle
from paper_2603_28768_amd import binding, synth

from cases import GATE_SHAPES, Case

pytestmark = pytest.mark.gpu

TOL = {"bf16": 1e-2, "f32": 1e-4}


def _np(t):
    return t.detach().float().cpu().numpy() if t.dtype.is_floating_point else t.detach().cpu().numpy()


# ----------------------------------------------------------------------- route

@pytest.mark.parametrize("T,E,k,quantum,renorm", [
    (256, 16, 2, None, True), (1000, 128, 8, None, True), (333, 256, 8, None, False),
    (97, 384, 8, None, True), (64, 100, 5, 0.5, True), (40, 7, 7, 1.0, False),
    (33, 1, 1, None, True), (31, 1000, 64, 0.25, True), (4096, 128, 8, None, True)])
def test_route_parity(torch_cuda, T, E, k, quantum, renorm):
    torch = torch_cuda
    print(f"route T={T} E={E} k={k} quantum={quantum} renorm={renorm}", flush=True)
    g = np.random.default_rng(T * 131 + E)
    l = (g.standard_normal((T, E)) * 2).astype(np.float32)
    if quantum:
        l = (np.round(l / quantum) * quantum).astype(np.float32)      # many exact ties
    ids, w = binding.route_topk(torch.from_numpy(l).cuda(), k, renorm)
    torch.cuda.synchronize()
    rid, rw = oracle.route(l, k, renorm)
    assert np.array_equal(_np(ids), rid)
    assert np.allclose(_np(w), rw, rtol=1e-5, atol=1e-30)


@pytest.mark.parametrize("E,ks", [(16, (1, 4, 5, 16)), (64, (4, 5, 14, 15)), (100, (3, 4, 13, 14)), (256, (2, 3, 13, 14)),
                                  (384, (1, 2, 13, 14)), (512, (1, 13, 14)), (23, (5, 6, 7))])
def test_route_on_both_sides_of_its_rule(torch_cuda, E, ks):
    # fewest and most picks that are gathered at once, and more picks than lanes with a score
    torch = torch_cuda
    g = np.random.default_rng(E)
    l = (g.standard_normal((500, E)) * 2).astype(np.float32)
    dev = torch.from_numpy(l).cuda()
    for k in ks:
        for renorm in (True, False):
            ids, w = binding.route_topk(dev, k, renorm)
            rid, rw = oracle.route(l, k, renorm)
            assert np.array_equal(_np(ids), rid)
            assert np.allclose(_np(w), rw, rtol=1e-5, atol=1e-30)


@pytest.mark.parametrize("E,k,most", [(8, 2, 0.82), (64, 2, 0.82), (128, 2, 0.94), (32, 12, 2.1)])
def test_route_gathers_only_where_that_is_sooner(torch_cuda, E, k, most):
    # time against 8 picks of 64 scores, which are gathered (62 us): gathered too, one or two picks took as
    # long (1.00, 0.99, 1.07; by rounds 0.68, 0.66, 0.83), and for more picks than lanes with a score
    # gathering came on top of the rounds (2.26; rounds alone 1.96)
    torch = torch_cuda
    T = 1 << 19

    def least(E, k):
        l = torch.randn((T, E), device="cuda:0")
        out = []
        for _ in range(8):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            binding.route_topk(l, k)
            a.record()
            for _ in range(20):
                binding.route_topk(l, k)
            b.record()
            torch.cuda.synchronize()
            out.append(a.elapsed_time(b) * 50)
        return min(out)

    us, eight = least(E, k), least(64, 8)
    print(f"  E={E} k={k}: {us:.1f} us, E=64 k=8: {eight:.1f} us, {us / eight:.2f}", flush=True)
    assert us <= most * eight


def test_route_reads_scores_that_are_not_16_byte_aligned(torch_cuda):
    # E % 4 == 0 lets the kernel read rows 16 bytes at a time, but only from a 16-byte aligned
    # base: a score matrix that starts 4 bytes into an allocation is read score by score
    torch = torch_cuda
    T, E, k = 300, 128, 8
    g = np.random.default_rng(77)
    l = (g.standard_normal((T, E)) * 2).astype(np.float32)
    flat = torch.empty(T * E + 1, dtype=torch.float32, device="cuda:0")
    view = flat[1:].view(T, E)
    view.copy_(torch.from_numpy(l))
    assert view.data_ptr() % 16 == 4 and view.is_contiguous()
    ids, w = binding.route_topk(view, k)
    rid, rw = oracle.route(l, k)
    assert np.array_equal(_np(ids), rid)
    assert np.allclose(_np(w), rw, rtol=1e-5, atol=1e-30)


# ---------------------------------------------------------------------- probes

def test_measurement_probes(torch_cuda):
    # the kernels of known work behind the benchmark's machine rates: the copy copies, the
    # other two run and report the work they were asked for
    torch = torch_cuda
    g = torch.Generator(device="cuda").manual_seed(3)
    a = torch.randint(0, 255, (1 << 20,), dtype=torch.uint8, device="cuda:0", generator=g)
    b = torch.zeros_like(a)
    binding.probe_copy(a, b)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    sink = torch.zeros(4 * 256, dtype=torch.float32, device="cuda:0")
    assert binding.probe_mfma_bf16(10, sink, blocks=4) == 4 * 4 * 10 * 4 * 2 * 32 * 32 * 16
    isink = torch.zeros(4 * 256, dtype=torch.int32, device="cuda:0")
    small = torch.full((64 << 10,), 3, dtype=torch.uint8, device="cuda:0")
    assert binding.probe_read(small, 3, isink, blocks=4) == 4 * 3 * (64 << 10)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(sink).all())
    # every thread XORs the same number of equal words: an even count cancels
    assert int(isink.abs().sum()) == 0
    with pytest.raises(binding.CraftError):
        binding.probe_read(small[:1000], 1, isink, blocks=4)          # not a multiple of 32 KiB


# ------------------------------------------------------------------------ load

@pytest.mark.parametrize("L,T,k,E,bt", [
    (1, 256, 2, 16, 256), (3, 1000, 8, 128, 256), (2, 17, 3, 9, 5), (2, 9000, 8, 256, 4500),
    (1, 20000, 8, 384, 20000), (4, 4096, 8, 4096, 1024), (1, 7, 1, 1, 2)])
def test_expert_load_parity(torch_cuda, L, T, k, E, bt):
    torch = torch_cuda
    print(f"load L={L} T={T} k={k} E={E} bt={bt}", flush=True)
    g = np.random.default_rng(L * 7 + T)
    pop = synth.popularity(E, 1.3, 0)
    ids = g.choice(E, size=(L, T, k), p=pop).astype(np.int32)
    got = binding.expert_load(torch.from_numpy(ids).cuda(), E, bt)
    torch.cuda.synchronize()
    want = oracle.expert_load(ids, E, bt)
    assert np.array_equal(_np(got), want)


def test_expert_load_on_a_zipf_trace(torch_cuda):
    # the multi-layer stack's trace shape at reduced length: 58 layers x 256 experts, top-8
    torch = torch_cuda
    L, E, k, T, bt = 58, 256, 8, 8192, 4096
    s = synth.trace_layer_exponents(L, 5)
    ids = np.stack([synth.routing_trace_layer(E, k, T, s[l], 5, l) for l in range(L)])
    print("zipf trace", ids.shape, flush=True)
    got = _np(binding.expert_load(torch.from_numpy(ids).cuda(), E, bt))
    torch.cuda.synchronize()
    want = oracle.expert_load(ids, E, bt)
    assert np.array_equal(got, want)
    assert np.all(got.sum(-1) == bt * k)


# ------------------------------------------------------------- gating network

# fp32 accumulation of H products against the checker's double sum: the running sum stays of
# the size of the scores (a few units), each of the H/16 accumulator updates rounds it at
# 2^-24 relative, so the error is a few 1e-7 of the score scale in practice and H * 2^-24 of
# it at the very worst; 1e-4 of the largest score leaves room for both and is still a
# hundred times finer than a dropped or doubled term.
GATE_TOL = 1e-4


@pytest.mark.parametrize("dtype,T,H,E", [
    ("bf16", 100, 72, 5),            # one ragged block of experts, ragged tokens and slab
    ("bf16", 517, 520, 24),
    ("bf16", 96, 256, 130),          # two blocks per wave
    ("bf16", 70, 128, 384),          # three
    ("bf16", 40, 64, 512),           # four
    ("bf16", 33, 8, 1000),           # eight, a single 16-byte chunk per row
    ("bf16", 33000, 64, 128),        # workgroups to spare: two token fragments each
    ("bf16", 300, 2048, 200),        # with a workspace: the contraction split eight ways
    ("bf16", 200, 1000, 100),        # split, ragged last slab and a last split shorter than the rest
    ("bf16", 200, 1024, 384),        # split with three blocks of experts per wave
    ("bf16", 129, 192, 60),          # the smallest batch past the thin tiles; as many slabs as stages
    ("bf16", 260, 456, 1000),        # four blocks of experts, the last one ragged
    ("bf16", 16500, 136, 150),       # two fragments of tokens without a workspace, ragged slab
    ("bf16", 8, 7168, 256),          # thin tiles, the contraction split eight ways
    ("bf16", 100, 1000, 100),        # thin, split, ragged slab, tokens and experts, two blocks of tokens
    ("bf16", 128, 2056, 384),        # thin, the last split shorter than the rest
    ("bf16", 17, 520, 40),           # thin, two splits of a ragged contraction
    ("f32", 50, 100, 12)])
def test_router_logits_parity(torch_cuda, dtype, T, H, E):
    cfg = synth.scaled(synth.CONFIGS["qwen3"], dtype=dtype, T=T, H=H, E=E)
    x, W = synth.activations(cfg), synth.gate_weights(cfg)
    xd, Wd = binding.to_device(x, dtype), binding.to_device(W, dtype)
    want = oracle.router_logits(x, W)
    U = np.zeros((E, H), dtype=np.float32)
    U[np.arange(E), np.arange(E) % H] = 1.0
    Ud = binding.to_device(U, dtype)
    ws = binding.router_logits_workspace(xd, Wd)
    print(f"  gate {dtype} T={T} H={H} E={E}: workspace {0 if ws is None else ws.numel()} bytes", flush=True)
    for workspace in ([None] if ws is None else [None, ws]):    # one workgroup per tile / split contraction
        got = _np(binding.router_logits(xd, Wd, workspace))
        assert got.shape == want.shape == (T, E)
        err = np.abs(got.astype(np.float64) - want).max()
        print(f"    max|ref|={np.abs(want).max():.3g} max|err|={err:.3g}", flush=True)
        assert err <= GATE_TOL * np.abs(want).max()
        # sums of a single term are exact: a gate of unit rows copies columns of x
        got = _np(binding.router_logits(xd, Ud, workspace))
        assert np.array_equal(got, x[:, np.arange(E) % H])
        # and the result depends on the arguments only
        assert np.array_equal(_np(binding.router_logits(xd, Wd, workspace)), _np(binding.router_logits(xd, Wd, workspace)))


@pytest.mark.parametrize("T,H,E", [shape for shape, *_ in GATE_SHAPES])      # (test_launch_shapes.py pins their tiles and splits)
def test_router_logits_of_every_tile_and_split(torch_cuda, T, H, E):
    cfg = synth.scaled(synth.CONFIGS["qwen3"], T=T, H=H, E=E)
    x, W = synth.activations(cfg), synth.gate_weights(cfg)
    xd, Wd = binding.to_device(x, "bf16"), binding.to_device(W, "bf16")
    want = oracle.router_logits(x, W)
    ws = binding.router_logits_workspace(xd, Wd)
    got = _np(binding.router_logits(xd, Wd, ws))
    err = np.abs(got.astype(np.float64) - want).max()
    print(f"  gate T={T} H={H} E={E}: max|ref|={np.abs(want).max():.3g} max|err|={err:.3g}", flush=True)
    assert err <= GATE_TOL * np.abs(want).max()
    assert np.array_equal(got, _np(binding.router_logits(xd, Wd, ws)))
    # a gate of unit rows copies columns of x, whichever part they are in
    U = np.zeros((E, H), dtype=np.float32)
    at = np.arange(E) * 7 % H
    U[np.arange(E), at] = 1.0
    assert np.array_equal(_np(binding.router_logits(xd, binding.to_device(U, "bf16"), ws)), x[:, at])


def test_router_logits_of_activations_past_the_memory_side_cache(torch_cuda):
    # one part, two blocks of experts that meet in one L2: a last eight of tiles that is not all there.  A gate of
    # unit rows copies columns of x
    torch = torch_cuda
    T, H, E = 16500, 7168, 300
    assert T * H * 2 > 220 << 20
    x = torch.randn(T, H, device="cuda:0").bfloat16()
    at = torch.arange(E, device="cuda:0") * 23 % H
    U = torch.zeros(E, H, dtype=torch.bfloat16, device="cuda:0")
    U[torch.arange(E, device="cuda:0"), at] = 1.0
    assert binding.router_logits_workspace(x, U) is None
    assert torch.equal(binding.router_logits(x, U), x[:, at].float())


def test_router_logits_empty_and_rejected(torch_cuda):
    torch = torch_cuda
    x = torch.zeros((0, 64), dtype=torch.bfloat16, device="cuda:0")
    W = torch.zeros((8, 64), dtype=torch.bfloat16, device="cuda:0")
    assert tuple(binding.router_logits(x, W).shape) == (0, 8)
    with pytest.raises(binding.CraftError):                       # bf16 rows must be whole 16-byte chunks
        binding.router_logits(torch.zeros((4, 12), dtype=torch.bfloat16, device="cuda:0"),
                              torch.zeros((8, 12), dtype=torch.bfloat16, device="cuda:0"))
    with pytest.raises(binding.CraftError):                       # more experts than the router takes
        binding.router_logits(torch.zeros((4, 8), dtype=torch.bfloat16, device="cuda:0"),
                              torch.zeros((1025, 8), dtype=torch.bfloat16, device="cuda:0"))


@pytest.mark.parametrize("name", ["qwen3", "kimi"])
def test_router_logits_full_size_feeds_the_router(torch_cuda, name):
    # full shapes; the checker affords a sample of the tokens.  The top-k decision is taken by
    # both sides on the same fp32 scores (the library's): ids bit-exact.
    torch = torch_cuda
    cfg = synth.CONFIGS[name]
    x, W = synth.activations(cfg), synth.gate_weights(cfg)
    xd, Wd = binding.to_device(x, cfg.dtype), binding.to_device(W, cfg.dtype)
    logits = binding.router_logits(xd, Wd, binding.router_logits_workspace(xd, Wd))
    toks = np.random.default_rng(5).choice(cfg.T, size=192, replace=False)
    toks = np.concatenate([toks, [0, cfg.T - 1]])
    want = oracle.router_logits(x[toks], W)
    got = _np(logits)
    err = np.abs(got[toks].astype(np.float64) - want).max()
    print(f"  gate {name}: max|ref|={np.abs(want).max():.3g} max|err|={err:.3g}", flush=True)
    assert err <= GATE_TOL * np.abs(want).max()
    ids, w = binding.route_topk(logits, cfg.k)
    ref_ids, ref_w = oracle.route(got, cfg.k)
    assert np.array_equal(_np(ids), ref_ids)
    assert np.allclose(_np(w), ref_w, rtol=1e-5, atol=1e-30)


@pytest.mark.parametrize("dtype,T,H,I,E,k,D,slots", [
    ("bf16", 600, 512, 384, 32, 4, 4, 4),
    ("bf16", 300, 2048, 64, 24, 2, 2, 2),        # the gate's contraction is split
    ("f32", 200, 96, 64, 12, 3, 2, 2)])
def test_forward_with_its_own_gating_network(torch_cuda, dtype, T, H, I, E, k, D, slots):
    # scores not handed in: the forward runs the gate first.  Its scores are the ones the
    # stand-alone call gives (same kernels, same workspace rule), and every decision after
    # them is taken on those fp32 scores by library and checker alike.
    torch = torch_cuda
    cfg = synth.scaled(synth.CONFIGS["qwen3"], dtype=dtype, T=T, H=H, I=I, E=E, k=k, D=D,
                       replica_slots=slots, zipf_s=1.2, profile_batches=2)
    case = Case(cfg)
    Wr = synth.gate_weights(cfg)
    Wrd = binding.to_device(Wr, dtype)
    packed = dtype == "bf16"
    for rank in range(D):
        own, x, _ = case.gpu_rank(rank, packed=packed, w_router=Wrd)
        out_own = own(x).clone()
        ids_own = own.debug["ids"].clone()
        logits = binding.router_logits(x, Wrd, binding.router_logits_workspace(x, Wrd))
        given, _, _ = case.gpu_rank(rank, packed=packed)
        out_given = given(x, logits)
        torch.cuda.synchronize()
        assert torch.equal(ids_own, given.debug["ids"]) and torch.equal(out_own, out_given)
        scores = _np(logits)
        want = oracle.router_logits(case.x, Wr)
        assert np.abs(scores - want).max() <= GATE_TOL * np.abs(want).max()
        ref = oracle.rank_forward(case.x, scores, cfg.k, case.slot_expert, case.rank_slot_off, rank,
                                  case.weights_of, True, None)
        assert np.array_equal(_np(ids_own), ref["ids"])
        assert np.array_equal(_np(own.debug["dest"]).reshape(-1), ref["dest"])
        assert own.result() == (ref["rows"], 0)
        err = np.abs(_np(out_own).astype(np.float64) - ref["out"]).max()
        assert err <= TOL[dtype] * np.abs(ref["out"]).max() + 1e-30


@pytest.mark.parametrize("tiled", [False, True])        # token rows copied by a small batch's dispatch, or not
@pytest.mark.parametrize("T,H,E,k,renorm", [
    (8, 7168, 256, 8, True),         # the most parts, in one trip
    (40, 4096, 128, 8, False),       # the parts are read a second time for the weights
    (100, 1000, 130, 4, True),       # scores read one by one, four parts
    (128, 2056, 100, 5, False),      # two chunks of 64 scores, ragged slab
    (300, 2048, 384, 8, True),       # several trips of three parts
    (129, 1024, 300, 14, False),     # several trips, arg-max rounds
    (1010, 456, 65, 4, False),       # two parts in one workgroup: nothing left to add
    (643, 2000, 129, 8, True), (600, 2056, 380, 6, False),   # four copies of eight parts
    (9200, 520, 129, 4, True),
    (60, 1024, 66, 1, True),
    # up to 32 tokens: by the dispatch launch itself
    (1, 1024, 64, 8, True), (32, 2048, 64, 20, False),       # up to 64 experts; picks in two places per lane
    (32, 4096, 128, 8, False), (9, 1024, 100, 4, True),      # up to 128
    (32, 1024, 130, 6, True), (32, 7168, 256, 8, False),     # up to 256; scores read one by one
    (32, 4096, 384, 8, True), (31, 2048, 383, 20, False)])   # up to 384: several trips of three parts
def test_forward_adds_up_the_parts_of_a_split_gate(torch_cuda, T, H, E, k, renorm, tiled):
    # the partial scores are added in the order the gate's own sum has, by the routing kernel or, up to 32
    # tokens, by the dispatch: the same bits as
    # the stand-alone scores handed in, and decisions and output as the checker takes them on those
    torch = torch_cuda
    cfg = synth.scaled(synth.CONFIGS["qwen3"], T=T, H=H, I=64, E=E, k=k, D=32, replica_slots=2, zipf_s=1.0, profile_batches=2)
    print("split gate", cfg, renorm, flush=True)
    case = Case(cfg)
    Wr = synth.gate_weights(cfg)
    Wrd = binding.to_device(Wr, "bf16")
    own, x, _ = case.gpu_rank(case.heaviest, packed=True, w_router=Wrd)
    given, _, _ = case.gpu_rank(case.heaviest, packed=True)
    own.args.renormalize = given.args.renormalize = int(renorm)
    if tiled:                                                           # the caller's own tile heights: never streamed
        own.args.tile_rows_gateup = given.args.tile_rows_gateup = 128
        assert own.tile_choice()[0] == 128
    elif T <= 32:
        assert own.tile_choice() == (64, 64, 0, 0)
    ws = binding.router_logits_workspace(x, Wrd)
    assert ws is not None and ws.numel() >= 2 * T * E * 4               # split
    logits = binding.router_logits(x, Wrd, ws)
    out_own, out_given = own(x).clone(), given(x, logits)
    torch.cuda.synchronize()
    for name in ("ids", "topk_w", "dest"):
        assert torch.equal(own.debug[name], given.debug[name])
    assert torch.equal(out_own, out_given)
    ref = oracle.rank_forward(case.x, _np(logits), k, case.slot_expert, case.rank_slot_off, case.heaviest, case.weights_of,
                              renorm, None)
    assert np.array_equal(_np(own.debug["ids"]), ref["ids"])
    assert np.allclose(_np(own.debug["topk_w"]), ref["w"], rtol=1e-5, atol=1e-30)
    assert np.abs(_np(out_own).astype(np.float64) - ref["out"]).max() <= TOL["bf16"] * np.abs(ref["out"]).max() + 1e-30


# --------------------------------------------------------------------- forward

def _row_units(case: Case, rank: int, heights):
    """Row ranges [a, b) (positions in the rank's row block) of everything the packed FFN
    schedules as a unit, for every way a busy slot's fragments may be cut into row-tiles of the
    given heights (full tiles and a remainder, or shared evenly between the tiles that a height in
    fifths of a fragment up to the given one asks for): the first and the last 32-row
    fragment of every row-tile of every slot with more than 64 rows, and every 32-row fragment
    of the slots with at most 64 rows (a tile of their own or a rider on a busy tile)."""
    p_lo, p_hi = case.rank_slot_off[rank], case.rank_slot_off[rank + 1]
    lo = int(case.slot_off[p_lo])
    units = []
    for p in range(p_lo, p_hi):
        a, n = int(case.slot_off[p]) - lo, int(case.slot_cnt[p])
        F = (n + 31) // 32
        if n == 0:
            continue
        if n <= 64:
            units += [(a + 32 * f, a + min(32 * f + 32, n)) for f in range(F)]
            continue
        for h in heights:
            f = h // 32
            cuts = [[min(i * f, F) for i in range((F + f - 1) // f + 1)]]
            for m in {-(-10 * F // tenths) for tenths in range(max(40, 10 * f - 8), 10 * f + 1, 2)}:
                cuts.append([i * F // m for i in range(m + 1)])
            for cut in cuts:
                for f0, f1 in zip(cut[:-1], cut[1:]):
                    units.append((a + 32 * f0, a + min(32 * f0 + 32, n)))
                    units.append((a + 32 * (f1 - 1), a + min(32 * f1, n)))
    return units


def _assert_units_compared(case: Case, rank: int, tokens, heights):
    """Every unit of the FFN's work on this rank has at least one row whose token is among the
    compared ones (all tokens when `tokens` is None)."""
    cfg = case.cfg
    p_lo, p_hi = case.rank_slot_off[rank], case.rank_slot_off[rank + 1]
    lo, hi = int(case.slot_off[p_lo]), int(case.slot_off[p_hi])
    seen = np.zeros(hi - lo, dtype=bool)
    d = case.dest.reshape(cfg.T, cfg.k)
    d = d if tokens is None else d[np.asarray(tokens)]
    d = d[(d >= lo) & (d < hi)]
    seen[d - lo] = True
    units = _row_units(case, rank, heights)
    missed = [u for u in units if not seen[u[0]:u[1]].any()]
    assert units and not missed, missed[:5]
    return len(units)


def _tokens_covering_units(case: Case, rank: int, heights, extra: int = 0):
    """A token for the first and for the last row of every unit (see _row_units), a few tokens
    with no row on the rank, and `extra` random ones."""
    cfg = case.cfg
    lo = int(case.slot_off[case.rank_slot_off[rank]])
    hi = int(case.slot_off[case.rank_slot_off[rank + 1]])
    toks = set()
    for a, b in _row_units(case, rank, heights):
        toks.add(int(case.src[lo + a]) // cfg.k)
        toks.add(int(case.src[lo + b - 1]) // cfg.k)
    d = case.dest.reshape(cfg.T, cfg.k)
    off = np.nonzero(~((d >= lo) & (d < hi)).any(1))[0]
    toks.update(int(t) for t in off[:2])
    if extra:
        toks.update(int(t) for t in np.random.default_rng(1).choice(cfg.T, size=extra, replace=False))
    return sorted(toks)


def _check_rank(torch, case: Case, rank: int, tokens=None, max_rows=0, packed=False, knobs=None, ref=None,
                cover=False):
    """One forward of `rank` through the C ABI against the checker: integer results everywhere,
    the output on `tokens` (None: every token).  `ref`: a checker result for the same rank and
    tokens computed earlier.  `cover`: also assert that the compared tokens reach every
    row-tile, cold slot and rider unit of the two grouped GEMMs as this launch cuts them."""
    cfg = case.cfg
    fwd, x, logits = case.gpu_rank(rank, max_rows, packed=packed)
    for name, value in (knobs or {}).items():          # tuning knobs of the packed FFN
        setattr(fwd.args, name, value)
    if cover:
        rg, rd, ride_g, ride_d = fwd.tile_choice()
        n = _assert_units_compared(case, rank, tokens, sorted({rg, rd}))
        print(f"  rank {rank}: row-tiles of {rg} (gate/up) and {rd} (down) rows, riders {ride_g}/{ride_d}; "
              f"{n} units of work all have compared rows", flush=True)
    out = fwd(x, logits)
    rows, ovf = fwd.result()
    if ref is None:
        ref = case.oracle_rank(rank, tokens)
    d = {k: _np(v) for k, v in fwd.debug.items()}
    assert np.array_equal(d["ids"], ref["ids"])
    assert np.allclose(d["topk_w"], ref["w"], rtol=1e-5, atol=1e-30)
    assert np.array_equal(d["counts"], ref["counts"])
    assert np.array_equal(d["slot_cnt"], ref["slot_cnt"])
    assert np.array_equal(d["slot_off"], ref["slot_off"])
    assert np.array_equal(d["dest"].reshape(-1), ref["dest"])
    assert np.array_equal(d["src"], ref["src"])
    assert rows == ref["rows"] and ovf == 0
    got = _np(out).astype(np.float64)
    if tokens is not None:
        got = got[np.asarray(tokens)]
    scale = np.abs(ref["out"]).max()
    err = np.abs(got - ref["out"]).max()
    print(f"  rank {rank} packed={packed}: rows={rows} max|ref|={scale:.4g} max|err|={err:.3g} "
          f"rel={err / max(scale, 1e-30):.3g}", flush=True)
    assert err <= TOL[cfg.dtype] * scale + 1e-30
    return _np(out).astype(np.float64), ref


def test_tiny_layer_all_ranks(torch_cuda):
    # the tiny fp32 layer: every rank's share executes; their sum is the un-sharded layer
    case = Case(synth.CONFIGS["tiny"])
    cfg = case.cfg
    print("tiny", case.rows, flush=True)
    total = np.zeros((cfg.T, cfg.H))
    ref_total = np.zeros((cfg.T, cfg.H))
    for g in range(cfg.D):
        out, ref = _check_rank(torch_cuda, case, g)
        total += out
        ref_total += ref["out"]
    assert np.abs(total - ref_total).max() <= TOL["f32"] * np.abs(ref_total).max()


@pytest.mark.parametrize("dtype,T,H,I,E,k,D,slots", [
    ("bf16", 600, 512, 384, 32, 4, 4, 4),        # several row tiles, ragged last tile
    ("bf16", 517, 520, 200, 24, 8, 3, 5),        # ragged K (520, 200) and ragged N (200)
    ("bf16", 96, 256, 128, 8, 2, 8, 0),          # one expert per rank, no replicas
    ("f32", 300, 100, 60, 12, 3, 2, 3),          # fp32 path with ragged everything
    ("bf16", 1500, 256, 192, 16, 8, 1, 0),       # single rank holds everything
    ("bf16", 40, 128, 64, 6, 1, 2, 2)])          # top-1
def test_reduced_layers_every_rank(torch_cuda, dtype, T, H, I, E, k, D, slots):
    cfg = synth.scaled(synth.CONFIGS["qwen3"], dtype=dtype, T=T, H=H, I=I, E=E, k=k, D=D,
                       replica_slots=slots, zipf_s=1.2, profile_batches=2)
    print("reduced", cfg, flush=True)
    case = Case(cfg)
    for g in range(D):
        _check_rank(torch_cuda, case, g)
        if dtype == "bf16":
            _check_rank(torch_cuda, case, g, packed=True)


def test_forward_is_reproducible_bit_for_bit(torch_cuda):
    torch = torch_cuda
    cfg = synth.scaled(synth.CONFIGS["qwen3"], T=700, H=256, I=256, E=32, D=4, replica_slots=4,
                       profile_batches=2)
    case = Case(cfg)
    fwd, x, logits = case.gpu_rank(case.heaviest, packed=True)
    a = fwd(x, logits).clone()
    da = {k: v.clone() for k, v in fwd.debug.items()}
    for _ in range(3):
        b = fwd(x, logits)
        torch.cuda.synchronize()
        assert torch.equal(a, b)
        for k, v in fwd.debug.items():
            assert torch.equal(da[k], v), k


def test_forward_replays_from_a_hip_graph(torch_cuda):
    # the forward is launches only (counters are cleared by a kernel, not a memset node), so it
    # can be captured; every replay, with eager work and synchronisations in between, has to
    # give the bits of the eager forward on the same inputs
    torch = torch_cuda
    cfg = synth.scaled(synth.CONFIGS["qwen3"], T=700, H=256, I=256, E=32, D=4, replica_slots=4,
                       profile_batches=2)
    case = Case(cfg)
    fwd, x, logits = case.gpu_rank(case.heaviest, packed=True)
    sx, sl = x.clone(), logits.clone()                 # the captured launches read these buffers
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for _ in range(2):
            fwd(sx, sl)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fwd(sx, sl)
    torch.cuda.synchronize()
    for shift in (0, 1, 37, 350):
        xs, ls = torch.roll(x, shift, 0), torch.roll(logits, shift, 0)   # other tokens, other routing
        want = fwd(xs, ls).clone()
        want_dest = fwd.debug["dest"].clone()
        torch.cuda.synchronize()
        sx.copy_(xs)
        sl.copy_(ls)
        fwd.out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(fwd.out, want), shift
        assert torch.equal(fwd.debug["dest"], want_dest), shift
    ref = case.oracle_rank(case.heaviest)
    sx.copy_(x)
    sl.copy_(logits)
    graph.replay()
    torch.cuda.synchronize()
    out = fwd.out.float().cpu().numpy().astype(np.float64)
    assert np.abs(out - ref["out"]).max() <= TOL[cfg.dtype] * np.abs(ref["out"]).max()


def test_one_expert_layer_is_the_dense_ffn(torch_cuda):
    # E = 1, k = 1: every token goes to the one expert with weight 1, which is how a dense
    # (shared) expert runs through the same entry point.  Alone on one rank the layer is the
    # plain SwiGLU FFN of every token; replicated on two ranks each takes every other token
    # (the i-th assignment goes to copy i mod 2) and the two outputs add up to it.
    for D, slots in ((1, 0), (2, 1)):
        cfg = synth.scaled(synth.CONFIGS["qwen3"], T=600, H=512, I=384, E=1, k=1, D=D,
                           replica_slots=slots, profile_batches=2)
        case = Case(cfg)
        dense = oracle.ffn_rows(case.x.astype(np.float32), *synth.expert_weights(cfg, 0))
        total = np.zeros_like(dense)
        for g in range(D):
            out, ref = _check_rank(torch_cuda, case, g, packed=True)
            assert ref["rows"] == cfg.T // D
            total += out
        assert np.abs(total - dense).max() <= TOL["bf16"] * np.abs(dense).max()


def test_rank_without_rows_and_unused_experts(torch_cuda):
    # strong skew on few tokens: some experts (and with D = E some ranks) get nothing
    cfg = synth.scaled(synth.CONFIGS["qwen3"], T=24, H=128, I=64, E=16, k=2, D=16,
                       replica_slots=0, zipf_s=3.0, profile_batches=1)
    case = Case(cfg)
    assert min(case.rows) == 0
    for g in (int(np.argmin(case.rows)), case.heaviest):
        out, _ = _check_rank(torch_cuda, case, g, packed=True)
        if case.rows[g] == 0:
            assert np.all(out == 0)


def test_packed_weights_layout(torch_cuda):
    # the packed stream against its stated layout, element by element
    torch = torch_cuda
    H, I = 72, 40                                   # ragged in every direction
    g = np.random.default_rng(5)
    mats = [synth.round_to_storage(g.standard_normal(s).astype(np.float32), "bf16")
            for s in ((I, H), (I, H), (H, I))]
    dev = [binding.to_device(m, "bf16") for m in mats]
    pgu, pdn = binding.pack_weights(*dev)
    torch.cuda.synchronize()
    pgu = synth.bf16_bits_to_f32(pgu.cpu().numpy().view(np.uint16))
    pdn = synth.bf16_bits_to_f32(pdn.cpu().numpy().view(np.uint16))
    Wg, Wu, Wd = mats

    def expect(groups, ksteps, row_of, K):
        # [32-wide step][column group][half][lane][8 values]
        out = np.zeros((ksteps, groups, 2, 64, 8), np.float32)
        for gi in range(groups):
            for s in range(ksteps):
                for h in range(2):
                    for l in range(64):
                        src = row_of(gi, h, l & 15)
                        k0 = 32 * s + 8 * (l >> 4)
                        if src is not None and k0 < K:
                            out[s, gi, h, l] = src[k0:k0 + 8]
        return out.reshape(-1)

    gu = expect(((I + 15) // 16 + 7) // 8 * 8, (H + 255) // 256 * 8,
                lambda gi, h, r: (Wu if h else Wg)[16 * gi + r] if 16 * gi + r < I else None, H)
    dn = expect(((H + 31) // 32 + 7) // 8 * 8, (I + 255) // 256 * 8,
                lambda gi, h, r: Wd[32 * gi + 16 * h + r] if 32 * gi + 16 * h + r < H else None, I)
    assert np.array_equal(pgu, gu) and np.array_equal(pdn, dn)


@pytest.mark.parametrize("H,I", [(1024, 136), (1032, 40), (2056, 1288), (8, 8)])
def test_packed_weights_layout_over_several_workgroups(torch_cuda, H, I):
    # parts of the contraction: exactly one, one and a ragged second, several on both sides
    g = np.random.default_rng(H + I)
    mats = [synth.round_to_storage(g.standard_normal(s).astype(np.float32), "bf16")
            for s in ((I, H), (I, H), (H, I))]
    pgu, pdn = (synth.bf16_bits_to_f32(p.cpu().numpy().view(np.uint16))
                for p in binding.pack_weights(*[binding.to_device(m, "bf16") for m in mats]))

    def fragments(W, rows, ksteps):                 # [rows / 16][ksteps][lane][8], zero padded
        P = np.zeros((rows, ksteps * 32), np.float32)
        P[:W.shape[0], :W.shape[1]] = W
        return P.reshape(rows // 16, 16, ksteps, 4, 8).transpose(0, 2, 3, 1, 4).reshape(rows // 16, ksteps, 64, 8)

    gu_rows, dn_rows = (I + 127) // 128 * 128, (H + 255) // 256 * 256
    gk, dk = (H + 255) // 256 * 8, (I + 255) // 256 * 8
    gu = np.stack([fragments(mats[0], gu_rows, gk), fragments(mats[1], gu_rows, gk)], axis=1)   # [group][half][step]
    assert np.array_equal(pgu, gu.transpose(2, 0, 1, 3, 4).reshape(-1))
    dn = fragments(mats[2], dn_rows, dk).reshape(dn_rows // 32, 2, dk, 64, 8)
    assert np.array_equal(pdn, dn.transpose(2, 0, 1, 3, 4).reshape(-1))


def test_empty_batch(torch_cuda):
    torch = torch_cuda
    cfg = synth.scaled(synth.CONFIGS["tiny"], T=0)
    W = np.ones((1, 1, cfg.E), dtype=np.int64)
    plan = binding.Plan(W, cfg.D, 0)
    ws = [torch.zeros((cfg.I, cfg.H), device="cuda") for _ in range(4)]
    wd = [torch.zeros((cfg.H, cfg.I), device="cuda") for _ in range(4)]
    fwd = binding.RankForward(plan, 0, 0, "f32", 0, cfg.H, cfg.I, cfg.k, ws, ws, wd)
    out = fwd(torch.empty((0, cfg.H), device="cuda"), torch.empty((0, cfg.E), device="cuda"))
    rows, ovf = fwd.result()
    assert tuple(out.shape) == (0, cfg.H) and rows == 0 and ovf == 0


def test_overflow_is_reported_not_computed(torch_cuda):
    cfg = synth.scaled(synth.CONFIGS["qwen3"], T=256, H=128, I=64, E=8, k=2, D=2,
                       replica_slots=0, profile_batches=1)
    case = Case(cfg)
    g = case.heaviest
    fwd, x, logits = case.gpu_rank(g, max_rows=case.rows[g] - 1)
    out = fwd(x, logits)
    rows, ovf = fwd.result()
    assert rows == case.rows[g] and ovf == 1
    assert np.all(_np(out) == 0)
    fwd2, x, logits = case.gpu_rank(g, max_rows=case.rows[g])      # exactly enough
    fwd2(x, logits)
    assert fwd2.result() == (case.rows[g], 0)


def test_forward_rejects_foreign_tables(torch_cuda):
    torch = torch_cuda
    cfg = synth.scaled(synth.CONFIGS["tiny"], T=64)
    case = Case(cfg)
    fwd, x, logits = case.gpu_rank(0)
    other = case.plan.upload_tables(0, 1)
    fwd.args.tables = other.data_ptr()                              # tables of another rank
    with pytest.raises(binding.CraftError):
        fwd(x, logits)
    fwd.args.tables = x.data_ptr()                                  # not a table buffer at all
    with pytest.raises(binding.CraftError):
        fwd(x, logits)
    # a buffer filled again for another rank counts for that rank only; filled again for the
    # same rank it stays good
    import ctypes
    mine = fwd.tables
    n = ctypes.c_size_t()
    lib = binding.lib()
    assert lib.craft_plan_tables_bytes(case.plan._h, 0, 1, ctypes.byref(n)) == 0
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert lib.craft_plan_tables_upload(case.plan._h, 0, 1, ctypes.c_void_p(mine.data_ptr()), n.value, stream) == 0
    fwd.args.tables = mine.data_ptr()
    with pytest.raises(binding.CraftError):
        fwd(x, logits)
    for _ in range(2):
        assert lib.craft_plan_tables_upload(case.plan._h, 0, 0, ctypes.c_void_p(mine.data_ptr()), n.value, stream) == 0
    ref = case.oracle_rank(0)
    out = fwd(x, logits)
    torch.cuda.synchronize()
    assert np.abs(_np(out).astype(np.float64) - ref["out"]).max() <= TOL[cfg.dtype] * np.abs(ref["out"]).max()


def test_rank_with_more_slots_than_the_tile_tables_in_lds(torch_cuda):
    # above 256 slots on a rank the FFN walks its tile tables in global memory
    cfg = synth.scaled(synth.CONFIGS["qwen3"], T=700, H=64, I=64, E=300, k=4, D=1, replica_slots=6,
                       zipf_s=1.1, profile_batches=2)
    case = Case(cfg)
    rows = case.slot_cnt
    assert len(rows) > 256 and (rows > 64).any() and ((rows > 0) & (rows <= 32)).any()
    outs = [_check_rank(torch_cuda, case, 0, packed=True, knobs=knobs)[0]
            for knobs in (dict(riders_gateup=-1, riders_down=-1),
                          dict(tile_rows_gateup=128, tile_rows_down=128, riders_gateup=1, riders_down=1))]
    assert np.array_equal(outs[0], outs[1])
    _check_rank(torch_cuda, case, 0, packed=False)


@pytest.mark.parametrize("dtype,T,H,E,k,renorm", [
    ("bf16", 1, 256, 8, 2, True),            # one token, one share of the columns
    ("bf16", 31, 4096, 64, 6, False),        # one chunk of scores, sixteen shares; weights from all scores
    ("bf16", 32, 520, 65, 4, True),          # scores read one by one
    ("f32", 32, 64, 128, 20, True),          # no rows copied, picks in two places per lane
    ("f32", 7, 100, 200, 8, False),
    ("bf16", 32, 2048, 384, 64, True),       # most experts and most picks
    ("bf16", 32, 256, 385, 8, True),         # more experts: routed by a launch of its own
    ("bf16", 33, 256, 64, 8, True)])         # two blocks: the same
def test_one_block_of_tokens_is_routed_by_the_dispatch(torch_cuda, dtype, T, H, E, k, renorm):
    torch = torch_cuda
    cfg = synth.scaled(synth.CONFIGS["qwen3"], dtype=dtype, T=T, H=H, I=64, E=E, k=k, D=3, replica_slots=3, zipf_s=1.0,
                       profile_batches=2)
    print("one block", cfg, renorm, flush=True)
    case = Case(cfg)
    fwd, x, logits = case.gpu_rank(case.heaviest, packed=dtype == "bf16")
    fwd.args.renormalize = int(renorm)
    ref = oracle.rank_forward(case.x, case.logits, k, case.slot_expert, case.rank_slot_off, case.heaviest, case.weights_of,
                              renorm, None)
    ids, w = binding.route_topk(logits, k, renormalize=renorm)      # the routing kernel's own
    for _ in range(2):
        out = fwd(x, logits)
        torch.cuda.synchronize()
        assert np.array_equal(_np(fwd.debug["ids"]), ref["ids"]) and torch.equal(fwd.debug["ids"], ids)
        assert torch.equal(fwd.debug["topk_w"], w)
        for name in ("dest", "src", "counts", "slot_cnt", "slot_off"):
            assert np.array_equal(_np(fwd.debug[name]).reshape(-1), ref[name]), name
        assert np.abs(_np(out).astype(np.float64) - ref["out"]).max() <= TOL[dtype] * np.abs(ref["out"]).max() + 1e-30


@pytest.mark.parametrize("T", [90, 1100, 2100])       # few blocks; prefixes in front
@pytest.mark.parametrize("slots", [1, 63, 64, 65])
def test_tile_tables_of_a_wave_of_slots(torch_cuda, T, slots):
    # a slot per lane up to 64 of them; slots of equal rows and, with 90 tokens, without any
    torch = torch_cuda
    cfg = synth.scaled(synth.CONFIGS["qwen3"], T=T, H=64, I=32, E=slots, k=min(2, slots), D=1, replica_slots=0,
                       zipf_s=1.3, profile_batches=2)
    _check_rank(torch, Case(cfg), 0, packed=True)


@pytest.mark.parametrize("dtype,H", [("bf16", 1016), ("bf16", 1024), ("bf16", 1032), ("bf16", 2056), ("f32", 508), ("f32", 512),
                                     ("f32", 516)])
def test_combine_of_rows_in_pieces(torch_cuda, dtype, H):
    # a wave takes 1024 (fp32: 512) columns of a row; a number of tokens that is no multiple of four
    torch = torch_cuda
    cfg = synth.scaled(synth.CONFIGS["qwen3"], dtype=dtype, T=201, H=H, I=40, E=12, k=6, D=2, replica_slots=1,
                       zipf_s=0.8, profile_batches=2)
    case = Case(cfg)
    for rank in range(2):
        _check_rank(torch, case, rank)


@pytest.mark.parametrize("dtype,T,H", [("bf16", 41, 1280), ("bf16", 41, 1288), ("f32", 41, 640), ("f32", 41, 644), ("bf16", 4097, 3080),
                                       ("bf16", 4097, 4608), ("bf16", 4097, 5128), ("f32", 4097, 1540)])
def test_combine_of_rows_in_longer_pieces(torch_cuda, dtype, T, H):
    # pieces of 1536 columns (fp32: 768): rows of one, three and four of them, whole and not, and a row too
    # long for one
    cfg = synth.scaled(synth.CONFIGS["qwen3"], dtype=dtype, T=T, H=H, I=40, E=12, k=6, D=2, replica_slots=1,
                       zipf_s=0.8, profile_batches=2)
    case = Case(cfg)
    toks = sorted(set(range(0, T, max(1, T // 40))) | {T - 1})
    for rank in range(2):
        _check_rank(torch_cuda, case, rank, tokens=toks)


def test_combine_in_several_launches(torch_cuda):
    # narrow rows, more tokens than the threads of one launch hold: every row of the result against a plain
    # fp32 product
    torch = torch_cuda
    T, H, I, E = (1 << 26) + 5, 8, 16, 4
    print("combine in launches", T, H, flush=True)
    plan = binding.Plan(np.full((1, 1, E), 8, dtype=np.int64), E, 0)
    lay = plan.layer(0)
    e = int(lay["slot_expert"][lay["rank_slot_off"][1]])
    g = torch.Generator(device="cuda:0").manual_seed(6)
    x = torch.empty((T, H), device="cuda:0", dtype=torch.bfloat16)
    for part in x.view(-1).split(1 << 26):
        part.copy_(torch.randn(part.numel(), generator=g, device="cuda:0"))
    w = [torch.randn(s, generator=g, device="cuda:0").bfloat16() * 0.5 for s in ((I, H), (I, H), (H, I))]
    picked = torch.randint(0, E, (T,), generator=g, device="cuda:0")
    logits = torch.zeros((T, E), device="cuda:0")
    logits.scatter_(1, picked[:, None], 4.0)
    rows = int((picked == e).sum())
    fwd = binding.RankForward(plan, 0, 1, "bf16", T, H, I, 1, [w[0]], [w[1]], [w[2]], max_rows=rows)
    fwd.out.fill_(float("nan"))
    out = fwd(x, logits)
    assert fwd.result() == (rows, 0)
    biggest, worst = 0.0, 0.0
    for t0 in range(0, T, 1 << 24):
        t1 = min(T, t0 + (1 << 24))
        xs = x[t0:t1].float()
        act = (torch.nn.functional.silu(xs @ w[0].float().t()) * (xs @ w[1].float().t())).bfloat16().float()
        ref = (act @ w[2].float().t()) * (picked[t0:t1] == e)[:, None]
        worst = max(worst, float((out[t0:t1].float() - ref).abs().nan_to_num(float("inf")).max()))
        biggest = max(biggest, float(ref.abs().max()))
    assert worst <= TOL["bf16"] * biggest


@pytest.mark.parametrize("T,E,k,D,slots", [
    # prefixes over chunks of 128 blocks, every workgroup derives the slots
    (3000, 160, 4, 4, 6),        # one chunk, three expert groups, a short last block
    (4100, 128, 8, 8, 16),       # two groups, one block more than a chunk
    (8192, 384, 8, 8, 24),       # six groups, two whole chunks
    (2000, 1024, 2, 16, 32),     # the most experts
    (8200, 72, 4, 2, 5),         # a third chunk of one block, ragged group
    (20000, 200, 3, 4, 9),       # five chunks of four groups, two blocks to a workgroup
    (1024, 40, 2, 2, 3),         # the largest batch dispatched from the blocks' counts alone
    (1025, 40, 2, 2, 3),         # the smallest with prefixes in front, ragged group
    (4096, 128, 8, 8, 16),       # two groups, one whole chunk
    (8192, 64, 3, 4, 20),        # one group, two whole chunks
    (8193, 64, 2, 2, 3),         # one group, a third chunk of one token
    (16385, 48, 2, 2, 3),        # two blocks to a workgroup, the last one alone
    (65536, 48, 1, 2, 3),        # the most chunks that a workgroup reads
    # the scan, by one workgroup per chunk and group
    (65537, 48, 1, 2, 3),        # the smallest such batch: nine chunks of one ragged group, one token in the last
    (65600, 16, 1, 2, 2),        # three blocks in the last
    (66000, 200, 3, 4, 9)])      # four groups
def test_dispatch_over_block_and_expert_shapes(torch_cuda, T, E, k, D, slots):
    # how the per-block counts are dealt to the waves depends on the number of 32-token blocks
    # and of 64-expert groups: integer results against the checker on every rank, narrow FFN
    cfg = synth.scaled(synth.CONFIGS["qwen3"], T=T, H=64, I=32, E=E, k=k, D=D, replica_slots=slots,
                       zipf_s=1.0, profile_batches=2)
    print("dispatch shapes", cfg, flush=True)
    case = Case(cfg)
    toks = list(range(0, T, max(1, T // 16)))
    for g in (0, D - 1):
        _check_rank(torch_cuda, case, g, tokens=toks, packed=True)


@pytest.mark.parametrize("T,E", [(64, 72), (96, 600), (128, 130), (160, 72), (225, 40), (256, 520), (290, 72), (420, 72), (1000, 72),
                                 (32768, 72), (41000, 40), (53000, 72), (65536, 72)])
def test_dispatch_over_numbers_of_totals(torch_cuda, T, E):
    # counts of 2 to 32 blocks, or of 8 to 16 chunks of blocks, added in eights, a four and single ones;
    # fewer and more experts than threads
    cfg = synth.scaled(synth.CONFIGS["qwen3"], T=T, H=64, I=32, E=E, k=3, D=2, replica_slots=3, zipf_s=1.0, profile_batches=1)
    print("numbers of totals", cfg, flush=True)
    case = Case(cfg)
    for g in (0, 1):
        _check_rank(torch_cuda, case, g, tokens=list(range(0, T, max(1, T // 16))), packed=True)


@pytest.mark.parametrize("T,E,k,D,slots", [
    # more than a workgroup of the direct dispatch keeps: scanned, whatever the batch
    (3000, 1024, 2, 64, 1100),   # a wave per group of experts
    (8192, 130, 2, 64, 2000),    # three groups, the whole chunk
    (9000, 1024, 2, 64, 1100),   # one workgroup per chunk and group, a ragged second chunk
    (300, 64, 2, 64, 2000),      # one whole group, few blocks
    (2000, 100, 2, 64, 2000),    # two groups, the second one ragged
    # one group of experts and more than 1536: scanned by a single workgroup
    (1025, 64, 2, 64, 1500),     # the smallest such batch
    (8192, 40, 3, 64, 1600)])    # the largest, ragged group
def test_dispatch_of_more_slots_than_a_workgroup_keeps(torch_cuda, T, E, k, D, slots):
    # the plan is the library's (its checker is slow at so many replicas)
    cfg = synth.scaled(synth.CONFIGS["qwen3"], T=T, H=64, I=32, E=E, k=k, D=D, replica_slots=slots, zipf_s=1.0)
    pop = synth.layer_popularity(cfg, 0)
    plan = binding.Plan(np.maximum(1, pop * 1e6).astype(np.int64)[None, None], D, slots)
    case = Case(cfg, plan=plan, pop=pop)
    assert len(case.slot_expert) > (2048 if E > 64 or T <= 1024 else 1536)
    for g in (0, D - 1):
        _check_rank(torch_cuda, case, g, tokens=list(range(0, T, T // 16)), packed=True)


@pytest.mark.parametrize("w8", [False, True])
@pytest.mark.parametrize("T,H,I,E,k,D,slots,zipf", [
    (240, 128, 192, 32, 4, 1, 0, 1.0),     # fewer busy tiles than units of the two-fragment slots
    (400, 128, 64, 48, 6, 1, 0, 1.5),      # more units than busy tiles: some cold tiles remain
    (900, 256, 320, 32, 4, 2, 2, 1.8)])    # three column tiles, replicas
def test_cold_slots_riding_with_busy_tiles(torch_cuda, T, H, I, E, k, D, slots, zipf, w8):
    # slots with at most 64 rows are carried by the tiles of busy slots or get tiles of their
    # own: every way of cutting the work gives the same bits, and those match the checker
    cfg = synth.scaled(synth.CONFIGS["qwen3"], T=T, H=H, I=I, E=E, k=k, D=D, replica_slots=slots,
                       zipf_s=zipf, profile_batches=2)
    case = Case(cfg, w8=w8)
    for g in range(D):
        rows = case.slot_cnt[case.rank_slot_off[g]:case.rank_slot_off[g + 1]]
        assert (rows > 64).any() and ((rows > 0) & (rows <= 32)).any()
        if D == 1:
            assert ((rows > 32) & (rows <= 64)).any()
        outs = []
        for knobs in (dict(riders_gateup=-1, riders_down=-1),
                      dict(tile_rows_gateup=128, tile_rows_down=160, riders_gateup=1, riders_down=1),
                      dict(tile_rows_gateup=224, tile_rows_down=224, riders_gateup=1, riders_down=-1),
                      dict(tile_rows_gateup=256, tile_rows_down=192, riders_gateup=1, riders_down=1)):
            print(" ", knobs, flush=True)
            outs.append(_check_rank(torch_cuda, case, g, packed=True, knobs=knobs)[0])
        for o in outs[1:]:
            assert np.array_equal(outs[0], o)


def test_block_ordered_tile_list_with_ragged_bands(torch_cuda):
    # more than two rounds of busy tiles over the CUs: the kernels walk every slot's tiles block
    # by block (bands of 8 row-tiles, blocks of 8 column tiles).  Four slots whose row-tile counts
    # are no multiples of 8 and 10 column tiles per slot in both GEMMs give ragged last bands and
    # a ragged last block of columns; every token is compared.
    cfg = synth.scaled(synth.CONFIGS["qwen3"], T=16000, H=2560, I=1280, E=4, k=1, D=1, replica_slots=0,
                       zipf_s=1.0, profile_batches=1)
    case = Case(cfg)
    rows = case.slot_cnt[case.rank_slot_off[0]:case.rank_slot_off[1]]
    fwd, _, _ = case.gpu_rank(0, packed=True)
    rg, rd, _, _ = fwd.tile_choice()
    for height, nt in ((rg, (cfg.I + 127) // 128), (rd, (cfg.H + 255) // 256)):
        row_tiles = [(int(r) + height - 1) // height for r in rows if r > 64]
        assert sum(row_tiles) * nt > 2 * 256 and any(m % 8 for m in row_tiles) and nt % 8
    print(f"  slot rows {rows.tolist()}, row-tiles of {rg}/{rd} rows", flush=True)
    _check_rank(torch_cuda, case, 0, packed=True, cover=True)


def test_packed_tiles_of_a_height_between_whole_fragments(torch_cuda):
    # six slots of some 63 fragments, three column tiles: the down GEMM takes twelve row-tiles a slot (even
    # heights of five or six whole fragments give thirteen or eleven), every token compared
    cfg = synth.scaled(synth.CONFIGS["qwen3"], T=12000, H=520, I=264, E=6, k=1, D=1, replica_slots=0, zipf_s=0.0,
                       profile_batches=2)
    case = Case(cfg)
    fwd, _, _ = case.gpu_rank(0, packed=True)
    assert fwd.tile_choice() == (160, 192, 0, 0)
    _check_rank(torch_cuda, case, 0, packed=True, cover=True)


@pytest.mark.parametrize("weights", ["packed", "e4m3", "rowmajor"])
@pytest.mark.parametrize("T,H,I,E,k,D,zipf,eval_zipf", [
    (1, 64, 32, 8, 1, 1, 1.0, 1.0),            # a single row; fewer slabs than waves
    (16, 72, 40, 8, 8, 2, 1.0, 1.0),           # exactly one fragment per slot; ragged K and N
    (17, 520, 200, 6, 6, 1, 1.0, 1.0),         # one row into the second fragment
    (33, 1544, 456, 6, 6, 1, 1.0, 1.0),        # one row into the third; a full ring with a remainder
    (64, 2112, 1288, 4, 4, 1, 1.0, 1.0),       # the most rows of one pass over the weights
    (200, 264, 136, 32, 4, 1, 0.0, 2.0),       # more rows than the plan expects: several passes
    (40, 128, 64, 300, 4, 1, 1.0, 1.0)])       # more slots than the tile tables in LDS hold
def test_small_batches_stream_the_weights(torch_cuda, T, H, I, E, k, D, zipf, eval_zipf, weights):
    cfg = synth.scaled(synth.CONFIGS["qwen3"], T=T, H=H, I=I, E=E, k=k, D=D, replica_slots=0, zipf_s=zipf,
                       profile_batches=4)
    print("small batch", cfg, weights, flush=True)
    case = Case(cfg, w8=weights == "e4m3")
    if eval_zipf != zipf:
        case = Case(cfg, plan=case.plan, pop=synth.popularity(E, eval_zipf, 1, 0), w8=case.w8)
        assert case.slot_cnt.max() > 64
    for g in range(D):
        fwd, _, _ = case.gpu_rank(g, packed=weights != "rowmajor")
        assert fwd.tile_choice() == (64, 64, 0, 0)
        _check_rank(torch_cuda, case, g, packed=weights != "rowmajor")


@pytest.mark.parametrize("H,I", [(8, 16), (64, 128), (128, 264), (200, 72), (256, 400), (520, 192)])
def test_rowmajor_tiles_of_every_height(torch_cuda, H, I):
    # one to nine slabs, ragged and whole, and slots on both sides of 32, 64 and 128 rows
    cfg = synth.scaled(synth.CONFIGS["qwen3"], T=1100, H=H, I=I, E=24, k=2, D=1, replica_slots=0, zipf_s=1.2, profile_batches=2)
    case = Case(cfg)
    rows = case.slot_cnt
    assert (rows > 128).any() and ((rows > 64) & (rows <= 128)).any() and ((rows > 32) & (rows <= 64)).any() and (rows <= 32).any()
    _check_rank(torch_cuda, case, 0, packed=False)


def _narrow_tiles(rows, K, N, gateup, num_cu=256):
    # the rule of ffn_bf16_kernel: whether the cold slots' tiles are a quarter as wide
    nt = -(-N // (128 if gateup else 256))
    busy, cold = sum(-(-r // 128) for r in rows if r > 64) * nt, sum(0 < r <= 64 for r in rows) * nt
    room = -busy % num_cu
    return busy + cold > num_cu and cold > room and cold * 1024 <= num_cu * K


@pytest.mark.parametrize("H,I,E,narrow", [
    (1608, 776, 40, (True, False)),  # the last quarters of gate/up's columns ragged or past the matrix; down many and short
    (1608, 1032, 40, (True, True)),  # and of down's
    (1792, 896, 40, (True, True)),   # whole tiles
    (1544, 776, 300, (True, False)),            # more slots than the tile tables in LDS
    (1544, 1288, 300, (False, True)),           # gate/up many and short
    (1288, 1736, 12, (False, False))])          # gate/up's cold tiles fit beside the last round of busy ones
def test_rowmajor_cold_slots_of_more_than_a_round(torch_cuda, H, I, E, narrow):
    cfg = synth.scaled(synth.CONFIGS["qwen3"], T=1100, H=H, I=I, E=E, k=2, D=1, replica_slots=0, zipf_s=1.0, profile_batches=2)
    case = Case(cfg)
    rows = case.slot_cnt
    assert (rows > 128).any() and ((rows > 32) & (rows <= 64)).any() and ((rows > 0) & (rows <= 32)).any()
    assert (I + 127) // 128 * sum(max(1, -(-r // 128)) for r in rows if r > 0) > 256
    assert (_narrow_tiles(rows, H, I, True), _narrow_tiles(rows, I, H, False)) == narrow
    _check_rank(torch_cuda, case, 0, packed=False)


@pytest.mark.parametrize("dtype,T,H,I,E", [
    ("bf16", 1100, 200, 72, 24), ("bf16", 40, 200, 72, 6), ("f32", 300, 52, 36, 8),
    ("bf16", 1100, 1608, 1032, 40)])                        # narrow tiles for the cold slots, in both GEMMs
def test_rowmajor_weights_at_any_element(torch_cuda, dtype, T, H, I, E):
    # contiguous views that start one element into an allocation: the same bits as aligned weights
    torch = torch_cuda
    cfg = synth.scaled(synth.CONFIGS["qwen3"], dtype=dtype, T=T, H=H, I=I, E=E, k=2, D=1, replica_slots=0, zipf_s=1.2, profile_batches=2)
    case = Case(cfg)
    narrow = (_narrow_tiles(case.slot_cnt, H, I, True), _narrow_tiles(case.slot_cnt, I, H, False))
    assert dtype == "f32" or narrow == (E == 40, E == 40)
    fwd, x, logits = case.gpu_rank(0)
    want = _np(fwd(x, logits).clone())

    def shifted(m):
        flat = torch.empty(m.numel() + 1, dtype=m.dtype, device=m.device)
        v = flat[1:].view(m.shape)
        v.copy_(m)
        assert v.data_ptr() % 16 == m.element_size()
        return v
    ws = [[shifted(m) for m in ms] for ms in fwd._weights]
    odd = binding.RankForward(case.plan, 0, 0, dtype, T, H, I, cfg.k, *ws)
    got = _np(odd(x, logits))
    assert np.array_equal(got, want)


def test_rowmajor_weights_with_tokens_past_4_gib(torch_cuda):
    # the gate/up GEMM leaves its 32-bit row offsets; the last tokens against a plain fp32 product
    torch = torch_cuda
    T, H, I, E, D = 310_000, 7168, 16, 64, 64
    plan = binding.Plan(np.full((1, 1, E), 8, dtype=np.int64), D, 0)
    e = int(plan.layer(0)["slot_expert"][plan.layer(0)["rank_slot_off"][5]])
    g = torch.Generator(device="cuda:0").manual_seed(5)
    x = torch.randn((T, H), generator=g, device="cuda:0", dtype=torch.bfloat16)
    w = [torch.randn(s, generator=g, device="cuda:0").bfloat16() * c for s, c in (((I, H), 0.01), ((I, H), 0.01), ((H, I), 0.25))]
    logits = torch.zeros((T, E), device="cuda:0")
    picked = torch.arange(T, device="cuda:0") % E
    logits[torch.arange(T, device="cuda:0"), picked] = 4.0
    fwd = binding.RankForward(plan, 0, 5, "bf16", T, H, I, 1, [w[0]], [w[1]], [w[2]])
    out = fwd(x, logits)
    assert fwd.result() == (int((picked == e).sum()), 0)
    toks = torch.nonzero(picked == e).flatten()[-100:]
    assert int(toks[0]) * H * 2 >= 1 << 32
    xs = x[toks].float()
    act = (torch.nn.functional.silu(xs @ w[0].float().t()) * (xs @ w[1].float().t())).bfloat16().float()
    ref = act @ w[2].float().t()
    assert (out[toks].float() - ref).abs().max() <= TOL["bf16"] * ref.abs().max()
    assert int(torch.count_nonzero(out[torch.nonzero(picked != e).flatten()[-100:]])) == 0


# -------------------------------------------------- full-size configurations

@pytest.mark.parametrize("name", ["qwen3", "dsv3", "kimi"])
def test_full_size_heaviest_rank_every_token(torch_cuda, name):
    # the launch configuration the benchmark times: full shapes, the heaviest rank's share, the
    # tile heights and rider switches the library picks by itself.  Integer results and the
    # output of EVERY token are compared (the checker does a rank's rows in seconds), so every
    # row of every row-tile, cold slot and rider unit of both GEMMs is looked at.
    import time
    cfg = synth.CONFIGS[name]
    print("full size", cfg, flush=True)
    case = Case(cfg)
    g = case.heaviest
    print(f"  rows per rank: max={max(case.rows)} mean={np.mean(case.rows):.0f} heaviest={g} "
          f"slot rows={case.slot_cnt[case.rank_slot_off[g]:case.rank_slot_off[g + 1]].tolist()}", flush=True)
    t0 = time.perf_counter()
    ref = case.oracle_rank(g)
    print(f"  checker: all {ref['rows']} rows, {cfg.T} tokens in {time.perf_counter() - t0:.1f} s", flush=True)
    _check_rank(torch_cuda, case, g, packed=True, ref=ref, cover=True)
    _check_rank(torch_cuda, case, g, packed=False, ref=ref)


# ------------------------------------------------------------- 8-bit expert weights

@pytest.mark.parametrize("rows,K,scale", [(7, 64, 1.0), (33, 520, 0.02), (5, 4096, 30.0), (1, 8, 1.0)])
def test_quantize_e4m3_parity(torch_cuda, rows, K, scale):
    torch = torch_cuda
    g = np.random.default_rng(rows * 1000 + K)
    W = synth.round_to_storage((g.standard_normal((rows, K)) * scale).astype(np.float32), "bf16")
    W[0, :8] = [0.0, -0.0, 1.0625, 1.1875, -1.0625, 448.0, 2.0 ** -10, 3 * 2.0 ** -10]   # zeros, ties, top
    if rows > 2:
        W[2] = 0.0                                                    # an all-zero row: scale 1
    codes, sc = binding.quantize_e4m3(binding.to_device(W, "bf16", "cuda:0"))
    want_c, want_s = oracle.quantize_e4m3(W)
    assert np.array_equal(sc.cpu().numpy(), want_s)
    assert np.array_equal(codes.cpu().numpy(), want_c)


@pytest.mark.parametrize("T,H,I,E,k,D,slots", [
    (600, 512, 384, 32, 4, 4, 4),          # several row tiles, ragged last tile
    (517, 520, 200, 24, 8, 3, 5),          # ragged K and N
    (40, 128, 64, 6, 1, 2, 2)])            # top-1, cold slots only
def test_reduced_layers_with_e4m3_weights(torch_cuda, T, H, I, E, k, D, slots):
    cfg = synth.scaled(synth.CONFIGS["qwen3"], T=T, H=H, I=I, E=E, k=k, D=D, replica_slots=slots,
                       zipf_s=1.2, profile_batches=2)
    case = Case(cfg, w8=True)
    for g in range(D):
        _check_rank(torch_cuda, case, g, packed=True)


def test_full_size_qwen3_with_e4m3_weights(torch_cuda):
    case = Case(synth.CONFIGS["qwen3"], w8=True)
    g = case.heaviest
    _check_rank(torch_cuda, case, g, packed=True, cover=True)          # every token


@pytest.mark.parametrize("H,I,scale", [
    (72, 40, 1.0),                   # one row block, ragged rows and steps, padding groups
    (264, 520, 0.02),                # ragged last row block
    (4096, 136, 30.0), (136, 2056, 1.0), (5000, 24, 1.0),      # 2, 4 and 8 step pairs per wave
    (8200, 16, 1.0),                 # rows that do not fit the registers
    (256, 64, 2.0 ** -75), (256, 64, 2.0 ** 90)])              # scales outside the reciprocal's range
def test_quantize_and_pack_in_one_pass_is_the_two_steps(torch_cuda, H, I, scale):
    # codes and scales are the checker's, and the packed bytes those of packing them
    torch = torch_cuda
    print(f"quantize+pack H={H} I={I} scale={scale}", flush=True)
    g = np.random.default_rng(H * 1000 + I)
    mats = [synth.round_to_storage((g.standard_normal(s) * scale).astype(np.float32), "bf16")
            for s in ((I, H), (I, H), (H, I))]
    mats[0][3] = 0.0
    mats[1][2, 5] = np.inf
    dev = [binding.to_device(m, "bf16") for m in mats]
    pgu, pdn = binding.pack_weights_e4m3(*dev)
    q = [binding.quantize_e4m3(m) for m in dev]
    want_gu, want_dn = torch.full_like(pgu, 0xAA), torch.full_like(pdn, 0xAA)
    ptr = binding._dev
    assert binding.lib().craft_pack_weights_e4m3(H, I, ptr(q[0][0]), ptr(q[1][0]), ptr(q[2][0]), ptr(q[0][1]), ptr(q[1][1]),
                                                 ptr(q[2][1]), ptr(want_gu), ptr(want_dn), binding._stream_ptr()) == 0
    torch.cuda.synchronize()
    for m, (codes, sc) in zip(mats, q):
        want_c, want_s = oracle.quantize_e4m3(m)
        finite = np.isfinite(m).all(axis=1)
        assert np.array_equal(sc.cpu().numpy(), want_s)
        assert np.array_equal(codes.cpu().numpy()[finite], want_c[finite])
    assert torch.equal(pgu, want_gu)
    assert torch.equal(pdn, want_dn)


@pytest.mark.parametrize("rows,tile_rows", [
    ([16, 40, 3, 5, 1, 30], 0),                                         # streamed
    *[([700, 300, 41, 20, 150, 260, 33, 9], r) for r in (128, 160, 192, 224, 256)]])        # tiles of every height, riders where they can be
def test_every_e4m3_code_through_the_gemms(torch_cuda, rows, tile_rows):
    # tokens and gate are chosen so that an output is 64 times one code: of the up matrix (experts 0, 2, 4 ..) or of the
    # down matrix.  The fifth and sixth also hold a NaN, which reaches everything that is multiplied by its row
    torch = torch_cuda
    H = I = 512
    E, T, dev = len(rows), sum(rows), "cuda:0"
    finite = torch.tensor([c for c in range(256) if c & 0x7F != 0x7F], dtype=torch.uint8, device=dev)
    value = finite.view(torch.float8_e4m3fn).float()
    n = torch.arange(512, device=dev)
    codes = finite[(n[:, None] + n[None, :]) % 254].contiguous()
    one = torch.zeros((512, 512), dtype=torch.uint8, device=dev)
    one[n, n] = 0x38                                                    # 1.0
    gate = torch.full((512, 512), 0x38, dtype=torch.uint8, device=dev)
    ones, g64 = torch.ones(512, device=dev), torch.full((512,), 64.0, device=dev)
    plan = binding.Plan(np.array(rows, dtype=np.int64)[None, None], 1, 0)
    lib, ptr, keep = binding.lib(), binding._dev, []

    def expert(e):
        up, down = (codes.clone(), one.clone()) if e % 2 == 0 else (one.clone(), codes.clone())
        if e == 4:
            up[5, 9] = 0x7F
        if e == 5:
            down[7, 11] = 0xFF
        m = torch.zeros((512, 512), dtype=torch.bfloat16, device=dev)
        gu, dn = binding.pack_weights_e4m3(m, m, m)                     # (buffers of the right size)
        assert lib.craft_pack_weights_e4m3(H, I, ptr(gate), ptr(up), ptr(down), ptr(g64), ptr(ones), ptr(ones), ptr(gu), ptr(dn),
                                           binding._stream_ptr()) == 0
        keep.append((up, down))
        return m, (gu, dn)
    ex = [expert(int(e)) for e in plan.layer(0)["slot_expert"]]
    fwd = binding.RankForward(plan, 0, 0, "bf16", T, H, I, 1, *[[m for m, _ in ex]] * 3, packed=[p for _, p in ex],
                              weight_format=binding.CRAFT_W_E4M3)
    fwd.args.tile_rows_gateup = fwd.args.tile_rows_down = tile_rows
    fwd.args.riders_gateup = fwd.args.riders_down = 1 if tile_rows else 0
    assert fwd.tile_choice()[:2] == ((tile_rows, tile_rows) if tile_rows else (64, 64))
    expert_of = torch.from_numpy(np.random.default_rng(1).permutation(np.repeat(np.arange(E), rows))).to(dev)
    logits = torch.where(n[None, :E] == expert_of[:, None], 5.0, -5.0).contiguous()
    h = torch.arange(T, device=dev) * 7 % H
    x = torch.zeros((T, H), dtype=torch.bfloat16, device=dev)
    x[torch.arange(T, device=dev), h] = 1.0
    out = fwd(x, logits).float()
    want = 64.0 * value[(n[None, :] + h[:, None]) % 254]
    want[expert_of == 4] = float("nan")
    want[expert_of == 5, 7] = float("nan")
    assert torch.equal(torch.isnan(out), torch.isnan(want))
    assert torch.equal(torch.nan_to_num(out, nan=0.0), torch.nan_to_num(want, nan=0.0))


@pytest.mark.parametrize("e4m3,I", [(False, (1 << 24) + 16), (True, (1 << 25) + 16)])
def test_packing_an_expert_of_very_many_columns(torch_cuda, e4m3, I):
    # a column group's place in the packed stream passes 2 GiB, the rows take more than one launch: the
    # first step of every group
    torch = torch_cuda
    H = 8
    print(f"packing H={H} I={I} e4m3={e4m3}", flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(I)
    up = torch.randn((I, H), generator=g, device="cuda:0").bfloat16()
    gate, down = -up, up.view(H, I)
    packed, _ = (binding.pack_weights_e4m3 if e4m3 else binding.pack_weights)(gate, up, down)
    groups, rows = (I // 16 + 7) // 8 * 8, I // 16
    per = groups * 2 * 64 * 8                             # elements of one step
    step = packed.view(torch.uint8 if e4m3 else torch.int16).reshape(-1)[:per].view(groups, 2, 64, 8)
    for half, m in enumerate((gate, up)):
        want = binding.quantize_e4m3(m)[0] if e4m3 else m.view(torch.int16)
        if e4m3:                                          # rows past the first launch, each with its own scale
            assert np.array_equal(_np(want[-4096:]), oracle.quantize_e4m3(_np(m[-4096:]))[0])
        assert torch.equal(step[:rows, half, :16], want.view(rows, 16, H))
        assert not step[:rows, half, 16:].any() and not step[rows:, half].any()


def test_router_logits_of_rows_past_32_bit_offsets(torch_cuda):
    # 256 rows of the gate take more than 4 GiB: a gate of unit rows copies columns of x
    torch = torch_cuda
    T, H, E = 140, (1 << 23) + 64, 256
    g = torch.Generator(device="cuda:0").manual_seed(3)
    x = torch.randn((T, H), generator=g, device="cuda:0").bfloat16()
    cols = H - 1 - 3 * torch.arange(E, device="cuda:0")
    W = torch.zeros((E, H), dtype=torch.bfloat16, device="cuda:0")
    W[torch.arange(E, device="cuda:0"), cols] = 1.0
    for workspace in (None, binding.router_logits_workspace(x, W)):
        assert torch.equal(binding.router_logits(x, W, workspace), x[:, cols].float())


@pytest.mark.parametrize("T,H,I", [(5, 256, (1 << 24) + 64), (3, (1 << 25) + 64, 136)])
def test_rowmajor_weights_of_rows_past_32_bit_offsets(torch_cuda, T, H, I):
    # the rows of one weight tile lie more than 4 GiB apart
    torch = torch_cuda
    print(f"long rows T={T} H={H} I={I}", flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(I)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda:0", dtype=torch.bfloat16)
    x, wg, wu, wd = rand(T, H) * H ** -0.5, rand(I, H), rand(I, H), rand(H, I) * I ** -0.5
    plan = binding.Plan(np.full((1, 1, 1), T, dtype=np.int64), 1, 0)
    fwd = binding.RankForward(plan, 0, 0, "bf16", T, H, I, 1, [wg], [wu], [wd])
    out = fwd(x, torch.zeros((T, 1), device="cuda:0")).float()
    # rows of the weights a part at a time: fp32 copies of the matrices would take most of the card
    part = max(1, (1 << 28) // H)
    act = torch.cat([torch.nn.functional.silu(x.float() @ a.float().t()) * (x.float() @ b.float().t())
                     for a, b in zip(wg.split(part), wu.split(part))], dim=1).bfloat16().float()
    part = max(1, (1 << 28) // I)
    ref = torch.cat([act @ a.float().t() for a in wd.split(part)], dim=1)
    assert (out - ref).abs().max() <= TOL["bf16"] * ref.abs().max()


def test_rowmajor_activation_is_the_same_in_small_and_large_batches(torch_cuda):
    # sums of one term, a unit down-projection: what comes out is silu(g) u rounded once, so the
    # streaming kernels and the tiles have to agree in every bit
    torch = torch_cuda
    E, rows, N = 8, 64, 2048
    g = torch.Generator(device="cuda:0").manual_seed(9)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda:0").bfloat16()
    T = E * rows
    x, wg, wu = (torch.zeros(s, dtype=torch.bfloat16, device="cuda:0") for s in ((T, N), (N, N), (N, N)))
    x[:, :2], wg[:, 0], wu[:, 1] = rand(T, 2), rand(N), rand(N)
    plan = binding.Plan(np.full((1, 1, E), rows, dtype=np.int64), 1, 0)
    fwd = binding.RankForward(plan, 0, 0, "bf16", T, N, N, 1, [wg] * E, [wu] * E, [torch.eye(N, device="cuda:0").bfloat16()] * E)
    logits = torch.zeros((T, E), device="cuda:0")
    logits[torch.arange(T), torch.arange(T) % E] = 4.0
    assert fwd.tile_choice() == (64, 64, 0, 0)
    streamed = fwd(x, logits).clone()
    fwd.args.workspace_bytes -= 1                          # the tiles, for which there is still room
    tiled = fwd(x, logits)
    assert int(torch.count_nonzero(tiled)) > T * N // 2
    assert torch.equal(streamed, tiled)


def test_rowmajor_weights_at_any_element_are_not_left_behind(torch_cuda):
    # loads of the next slab have to travel while one is multiplied: 1.6 to 1.9 times the time of aligned
    # weights, one slab at a time it was more than 4 times
    torch = torch_cuda
    E, rows, H, I = 17, 100, 4096, 1536
    g = torch.Generator(device="cuda:0").manual_seed(2)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda:0").bfloat16()
    plan = binding.Plan(np.full((1, 1, E), rows, dtype=np.int64), 1, 0)
    T = E * rows
    x, logits = rand(T, H), torch.zeros((T, E), device="cuda:0")
    logits[torch.arange(T), torch.arange(T) % E] = 4.0
    times = []
    for start in (0, 1):
        ws = [[], [], []]
        for _ in range(E):
            for out, s in zip(ws, ((I, H), (I, H), (H, I))):
                out.append(rand(s[0] * s[1] + 8)[start:start + s[0] * s[1]].view(s))
        fwd = binding.RankForward(plan, 0, 0, "bf16", T, H, I, 1, *ws)
        assert fwd.tile_choice() == (128, 128, 0, 0)
        best = []
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(5):
                fwd(x, logits)
            b.record()
            torch.cuda.synchronize()
            best.append(a.elapsed_time(b))
        times.append(min(best))
    print(f"  aligned {times[0] * 200:.0f} us, one element past it {times[1] * 200:.0f} us", flush=True)
    assert times[1] <= 3.0 * times[0]
