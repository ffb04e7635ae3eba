"""GPU tests of kernel choices at the sizes where they can go wrong: edges of
tiles, remainders, the smallest and largest of a rule's range, against the
fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import vfm_oracle as O
from paper_2606_09643_amd import binding as B
from paper_2606_09643_amd import runner as R
from paper_2606_09643_amd import workloads as wl
from tests.gpu_common import log, oracle_layer_rows, oracle_plan, seeded_rows, set_rows, tol
from tests.helpers import np64, oracle_weights, spec_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("idx,d,pool,hidden", [(2, 64, "first", 64), (2, 768, "last", 0), (5, 4096, "last", 128),
                                               (3, 1024, "mean", 0), (1, 256, "first", 64)])
def test_heads_output_and_request_remainders(idx, d, pool, hidden):
    """Head widths around the 16-output blocks (1, 15, 16, 17, 250), tasks of
    0, 1, 16, 17, 65 and 130 requests (groups of 16, up to 64 in one pass),
    linear and MLP heads side by side, one-row and mean pooling."""
    w = wl.WORKLOADS[idx].replace(d=d, n_heads=d // 64, head_dim=64, n_tasks=6, pool=pool, mode="prefill")
    n_out = np.array([17, 250, 1, 16, 15, 33], np.int32)
    counts = [65, 1, 17, 16, 130, 0]
    r = np.random.default_rng(5)
    task = r.permutation(np.repeat(np.arange(6), counts)).astype(np.int32)
    batch = wl.Batch(task, r.integers(1, 4, size=len(task)).astype(np.int32), None)
    g = torch.Generator(device="cuda").manual_seed(3)
    t_ = lambda *shape, std: (torch.randn(*shape, generator=g, device="cuda") * std).to(w.torch_dtype)  # noqa: E731
    mlp = [hidden > 0 and t % 2 == 0 for t in range(6)]
    Ws = [t_(int(n), hidden if m else d, std=(hidden if m else d) ** -0.5) for n, m in zip(n_out, mlp)]
    bs = [t_(int(n), std=0.1) if t != 3 else None for t, n in enumerate(n_out)]
    W1 = [t_(hidden, d, std=d ** -0.5) if m else None for m in mlp] if hidden else None
    b1 = [t_(hidden, std=0.1) if m else None for m in mlp] if hidden else None
    tab = B.HeadTable(n_out, Ws, bs, R._POOL[pool], W1s=W1, b1s=b1, hidden=hidden)
    final = wl.final_norm(w, "cuda")
    pb = B.Batch(batch.task_id, batch.seq_len, 6, n_out=n_out)
    x = torch.empty(pb.T, d, device="cuda")
    rows = seeded_rows(pb.T, d, 11)
    set_rows(x, rows)
    cfg = R.cfg_for(w)
    ws = torch.empty(B.vfm_workspace_size(cfg, pb.c), dtype=torch.uint8, device="cuda")
    out = torch.full((pb.total_outputs,), float("nan"), device="cuda")
    log(f"heads d={d} pool={pool} hidden={hidden}")
    B.vfm_head_forward(cfg, final["w"], final["b"], tab.c, pb.c, x, out, ws)
    got = out.cpu().numpy()
    pl = oracle_plan(w, batch, n_out)
    cu, off, spec = pl["cu_seqlens"], pl["logit_off"], spec_of(w)
    fb = np64(final["b"]) if final["b"] is not None else None
    ref = np.empty(len(got))
    for p, i in enumerate(pl["order"]):
        t = int(pl["task"][p])
        v = O.pool(O.final(spec, np64(final["w"]), fb, rows[int(cu[p]):int(cu[p + 1])]), pool)
        b = np64(bs[t]) if bs[t] is not None else np.zeros(int(n_out[t]))
        ref[off[i]:off[i + 1]] = (O.head_mlp(v, np64(W1[t]), np64(b1[t]), np64(Ws[t]), b) if mlp[t]
                                  else O.head(v, np64(Ws[t]), b))
    err = np.abs(got - ref).max() / np.abs(ref).max()
    log(f"  max rel err {err:.3e}")
    assert err < tol(w)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("pool", ["mean", "first"])
def test_heads_of_a_table_larger_than_the_batch(pool, dtype):
    """More tasks than requests: first and last ids, neighbouring ones, several
    requests of one task, MLP and linear heads, a head without outputs."""
    w = wl.WORKLOADS[2].replace(n_tasks=2500, pool=pool, dtype=dtype)
    hidden, ids, counts = 64, [0, 1, 700, 701, 1024, 2499], [3, 1, 1, 18, 2, 1]
    n_out = np.zeros(w.n_tasks, np.int32)
    n_out[ids] = [17, 1, 250, 33, 0, 1000]
    r = np.random.default_rng(5)
    task = r.permutation(np.repeat(ids, counts)).astype(np.int32)
    batch = wl.Batch(task, r.integers(1, 4, size=len(task)).astype(np.int32), None)
    g = torch.Generator(device="cuda").manual_seed(3)
    t_ = lambda *shape, std: (torch.randn(*shape, generator=g, device="cuda") * std).to(w.torch_dtype)  # noqa: E731
    Ws, W1, b1 = [None] * w.n_tasks, [None] * w.n_tasks, [None] * w.n_tasks
    for t in ids:
        if t % 2:
            W1[t], b1[t] = t_(hidden, w.d, std=w.d ** -0.5), t_(hidden, std=0.1)
        if n_out[t]:
            k = hidden if t % 2 else w.d
            Ws[t] = t_(int(n_out[t]), k, std=k ** -0.5)
    tab = B.HeadTable(n_out, Ws, [None] * w.n_tasks, R._POOL[pool], W1s=W1, b1s=b1, hidden=hidden)
    final, pb = wl.final_norm(w, "cuda"), B.Batch(batch.task_id, batch.seq_len, w.n_tasks, n_out=n_out)
    rows, cfg = seeded_rows(pb.T, w.d, 11), R.cfg_for(w)
    x = torch.empty(pb.T, w.d, device="cuda")
    set_rows(x, rows)
    ws = torch.empty(B.vfm_workspace_size(cfg, pb.c), dtype=torch.uint8, device="cuda")
    out = torch.full((pb.total_outputs,), float("nan"), device="cuda")
    log(f"heads of 2500 tasks pool={pool} {dtype}")
    B.vfm_head_forward(cfg, final["w"], final["b"], tab.c, pb.c, x, out, ws)
    got = out.cpu().numpy()
    pl, spec = oracle_plan(w, batch, n_out), spec_of(w)
    cu, off = pl["cu_seqlens"], pl["logit_off"]
    ref = np.empty(len(got))
    for p, i in enumerate(pl["order"]):
        t = int(pl["task"][p])
        v = O.pool(O.final(spec, np64(final["w"]), np64(final["b"]), rows[int(cu[p]):int(cu[p + 1])]), pool)
        z = np.zeros(int(n_out[t]))
        if n_out[t]:
            ref[off[i]:off[i + 1]] = (O.head_mlp(v, np64(W1[t]), np64(b1[t]), np64(Ws[t]), z) if t % 2
                                      else O.head(v, np64(Ws[t]), z))
    err = np.abs(got - ref).max() / np.abs(ref).max()
    log(f"  max rel err {err:.3e}")
    assert err < tol(w)


def _us(run, n=20):
    """Median time of run() on the GPU, microseconds."""
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2 * n)]
    for _ in range(3):
        run()
    for i in range(n):
        ev[2 * i].record()
        run()
        ev[2 * i + 1].record()
    torch.cuda.synchronize()
    return float(np.median([ev[2 * i].elapsed_time(ev[2 * i + 1]) for i in range(n)])) * 1e3


def test_heads_time_follows_the_batch():
    """One request's head costs about the same among 8192 tasks of 1000 outputs
    as among 16 (a grid over the whole table took 18 times as long)."""
    w = wl.WORKLOADS[2]
    W = torch.randn(1000, w.d, device="cuda").to(w.torch_dtype)
    final, cfg, t = wl.final_norm(w, "cuda"), R.cfg_for(w), {}
    for n in (16, 8192):
        n_out = np.full(n, 1000, np.int32)
        tab = B.HeadTable(n_out, [W] * n, [None] * n, R._POOL["first"])
        pb = B.Batch(np.array([n // 2], np.int32), np.ones(1, np.int32), n, n_out=n_out)
        x, out = torch.randn(1, w.d, device="cuda"), torch.empty(1000, device="cuda")
        ws = torch.empty(B.vfm_workspace_size(cfg, pb.c), dtype=torch.uint8, device="cuda")
        log(f"head among {n} tasks")
        t[n] = _us(lambda: B.vfm_head_forward(cfg, final["w"], final["b"], tab.c, pb.c, x, out, ws))
        log(f"  {t[n]:.1f} us")
    assert t[8192] < 4 * t[16], t


def _rows_of(w, model, task, length, seeds):
    """Layer outputs of requests whose input rows follow from their own seeds,
    in arrival order (one list entry per request)."""
    task, length = np.asarray(task, np.int32), np.asarray(length, np.int32)
    pb = R.make_batch(w, wl.Batch(task, length, None), None)
    order = np.argsort(task, kind="stable")
    x = torch.empty(pb.T, w.d, device="cuda")
    set_rows(x, np.concatenate([seeded_rows(int(length[i]), w.d, seeds[i]) for i in order]))
    ws = torch.empty(B.vfm_workspace_size(model.cfg, pb.c, model.lora_c(0)), dtype=torch.uint8, device="cuda")
    B.vfm_layer_forward(model.cfg, model.c_layers[0], model.lora_c(0), pb.c, x, workspace=ws)
    got, cu = x.cpu(), np.concatenate([[0], np.cumsum(length[order])])
    out = [None] * len(task)
    for p, i in enumerate(order):
        out[i] = got[int(cu[p]):int(cu[p + 1])]
    return out


@pytest.mark.parametrize("idx,d,d_ff,ranks", [(4, 2048, 5504, [16, 0, 8]), (4, 1024, 2816, [8, 64, 0]),
                                              (2, 768, 3072, [16, 0, 8]), (3, 1024, 2816, [0, 40, 8])])
@pytest.mark.parametrize("lens", [[1, 40, 23], [64, 1, 63], [130, 64, 65], [200, 300, 523]])
def test_small_batch_rows_same_in_any_tile(idx, d, d_ff, ranks, lens):
    """Batches below the small-batch threshold: a request's rows are the same
    bits alone and in batches that take another row tile (64, 128 or 256 rows
    of the split-K GEMM, 64 or 128 of the direct one)."""
    w = wl.WORKLOADS[idx].replace(d=d, n_heads=d // 128 if idx == 4 else d // 64, d_ff=d_ff, n_tasks=3,
                                  lora_targets=wl.PROJ if idx == 4 else ("q", "v", "o", "up", "down"))
    model = R.Model(w, n_layers=1, ranks=np.asarray(ranks, np.int32), b_std=0.05)
    log(f"small batch {w.name} d={d} lens={lens}")
    whole = _rows_of(w, model, [2, 0, 1], lens, [5, 6, 7])
    for i, t in enumerate([2, 0, 1]):
        alone = _rows_of(w, model, [t], [lens[i]], [5 + i])[0]
        assert torch.equal(alone, whole[i]), f"request {i} of {lens}"


_SMALL, _MID = ([1, 2, 1, 3, 1], [70, 30, 1, 40, 200]), [700, 300, 100, 17, 400]


@pytest.mark.parametrize("idx,d,hd,d_ff,ranks,lens", [
    *((*c, n) for n in _SMALL for c in (
        (2, 768, 64, 3072, [16, 8, 16, 0, 8]), (3, 1024, 64, 2816, [64, 8, 16, 0, 40]),
        (4, 1024, 128, 960, [16, 16, 8, 0, 8]), (4, 1024, 128, 960, [32, 8, 32, 16, 24]),
        (4, 1024, 128, 960, [48, 64, 8, 0, 16]), (4, 2048, 128, 5504, [16, 8, 16, 0, 8]))),
    (2, 768, 64, 3072, [16, 8, 16, 0, 8], _MID), (3, 1024, 64, 2816, [64, 8, 16, 0, 40], _MID),
    (4, 1024, 64, 960, [16, 16, 8, 0, 8], _MID), (4, 1024, 64, 960, [48, 64, 8, 0, 16], _MID),
    (2, 768, 64, 3072, [16, 8, 16, 0, 8], [1500, 800, 300, 1200, 900]),       # O and down alone: 128-row tiles
    (2, 768, 64, 3072, [64, 8, 16, 0, 40], [1500, 800, 300, 1200, 900])])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_broken_adapter_stays_with_its_task(idx, d, hd, d_ff, ranks, lens, bad):
    """Batches on the 64- and 128-row tiles and on the split path: a task whose
    expand factors hold an infinity or a NaN spoils its own requests only; every
    other request keeps its bits, in tiles that hold rows of both, LoRA steps of
    one run and of several."""
    w = wl.WORKLOADS[idx].replace(d=d, n_heads=d // hd, head_dim=hd, d_ff=d_ff, n_tasks=5,
                                  lora_targets=wl.PROJ if idx == 4 else ("o", "down") if sum(lens) > 2000
                                  else ("q", "k", "v", "o", "up", "down"))
    model = R.Model(w, n_layers=1, ranks=np.asarray(ranks, np.int32), b_std=0.05)
    log(f"broken adapter {w.name} d={d} lens={lens} ranks={ranks} {bad}")
    whole = _rows_of(w, model, [3, 0, 2, 1, 4], lens, [5, 6, 7, 8, 9])
    for p, B_t in model.adapters[0].B.items():
        B_t[2, ::7] = bad
    got = _rows_of(w, model, [3, 0, 2, 1, 4], lens, [5, 6, 7, 8, 9])
    assert not got[2].isfinite().any()
    for i in (0, 1, 3, 4):
        assert whole[i].isfinite().all() and torch.equal(whole[i], got[i]), f"request {i}"


@pytest.mark.parametrize("idx,more", [(2, [1024 - 197]), (2, [5000]), (3, [1000]), (3, [9000])])
def test_large_batch_rows_same_in_any_tile(idx, more):
    """From the threshold on: the same bits from the 64- and 128-row tiles of
    batches that cannot fill the chip and the 256-row ones of batches that can."""
    w = wl.WORKLOADS[idx].replace(n_tasks=3, lora_targets=("q", "k", "v", "o", "up", "down"))
    model = R.Model(w, n_layers=1, ranks=np.asarray([16, 0, 8], np.int32), b_std=0.05)
    split = lambda n: [256] * (n // 256) + ([n % 256] if n % 256 else [])   # noqa: E731
    log(f"large batch {w.name} beside {more} rows")
    base = _rows_of(w, model, [1] + [0] * len(split(20000)), [197] + split(20000), [9] + list(range(20, 20 + 79)))[0]
    got = _rows_of(w, model, [1] + [2] * len(split(more[0])), [197] + split(more[0]),
                   [9] + list(range(200, 200 + len(split(more[0])))))[0]
    assert torch.equal(base, got)


@pytest.mark.parametrize("idx,hd,lens,ranks", [
    (1, 64, [3, 70, 20], [8, 16, 64]), (2, 64, [3, 70, 20], [8, 16, 64]), (2, 64, [900, 700, 1000], [16, 16, 8]),
    (2, 64, [900, 700, 1000], [8, 40, 8]), (4, 128, [3, 20, 10], [8, 16, 32]), (4, 128, [60, 20, 90], [8, 16, 64]),
    (4, 128, [300, 20, 90], [16, 16, 8])])
def test_task_with_bare_projections(idx, hd, lens, ranks):
    """A task that has an adapter for some projections of the table only (NULL
    entries for the others), on every path: the fp32 kernels, the small and the
    large tiles, the split shrink in the GEMM's launch and in its own."""
    more = {4: dict(d=1536, d_ff=1856)}.get(idx, {})
    w = wl.WORKLOADS[idx].replace(n_tasks=3, head_dim=hd, **more)
    targets = wl.PROJ if w.family == "decoder" else ("q", "k", "v", "o", "up", "down")
    w = w.replace(n_heads=w.d // hd, lora_targets=targets)
    has = {0: targets, 1: targets[::2], 2: targets[1:3]}
    model = R.Model(w, n_layers=1, ranks=np.asarray(ranks, np.int32), b_std=0.03)
    ad = model.adapters[0]
    factors = {p: ([ad.a(p, t) if p in has[t] else None for t in range(3)],
                   [ad.b(p, t) if p in has[t] else None for t in range(3)]) for p in targets}
    model.lora[0] = B.LoraTable(3, ad.rank, ad.scale, factors, max_rank=ad.max_rank)
    log(f"bare projections {w.name} lens={lens}")
    got = _rows_of(w, model, [1, 0, 2], lens, [5, 6, 7])
    worst = 0.0
    for i, t in enumerate([1, 0, 2]):
        rows = seeded_rows(lens[i], w.d, 5 + i)
        only = {p: (np64(ad.a(p, t)), np64(ad.b(p, t)), float(ad.scale[t])) for p in has[t]}
        y = O.layer(spec_of(w), oracle_weights(model.layers[0]), only, rows, pos=np.arange(lens[i]))[0]
        worst = max(worst, O.row_rel_error(got[i].double().numpy(), y))
    log(f"  max rel err {worst:.3e}")
    assert worst < tol(w)


def _layer_case(w, task, length, ranks, seed=1, b_std=0.05):
    batch = wl.Batch(np.asarray(task, np.int32), np.asarray(length, np.int32), None)
    model = R.Model(w, n_layers=1, ranks=np.asarray(ranks, np.int32), b_std=b_std, seed=seed)
    pb = R.make_batch(w, batch, None)
    rows = seeded_rows(pb.T, w.d, 7)
    x = torch.empty(pb.T, w.d, device="cuda")
    ws = torch.empty(B.vfm_workspace_size(model.cfg, pb.c, model.lora_c(0)), dtype=torch.uint8, device="cuda")
    pl = oracle_plan(w, batch)

    def run(x):
        set_rows(x, rows)
        B.vfm_layer_forward(model.cfg, model.c_layers[0], model.lora_c(0), pb.c, x, workspace=ws)
        return x.double().cpu().numpy()

    return model, pl, rows, run(x)


def _check_layer(w, model, pl, rows, got, reqs):
    ref = oracle_layer_rows(w, oracle_weights(model.layers[0]), model.adapters[0], pl, rows, reqs)
    cu, worst = pl["cu_seqlens"], 0.0
    for p in reqs:
        worst = max(worst, O.row_rel_error(got[int(cu[p]):int(cu[p + 1])], ref[p][0]))
    log(f"  max rel err {worst:.3e}")
    assert worst < tol(w)


@pytest.mark.parametrize("lens,family,hd,d_ff", [
    ([1], "encoder", 64, 64), ([31, 1, 2], "encoder", 64, 320), ([33, 64, 65], "encoder", 128, 1024),
    ([200, 16, 17, 1], "encoder", 64, 2048), ([130, 7, 64], "decoder", 128, 192),
    ([1100, 400, 700, 2000, 5], "encoder", 64, 1024)])
def test_f32_layer_tiles(lens, family, hd, d_ff):
    """The fp32 layer at the edges of its 32- and 64-row tiles, 16-query
    attention groups and 16 / 32 / 64-rank shrink sub-tiles (both GEMM tile
    shapes; the last batch takes the 64x64 one), d_ff not a multiple of 128."""
    w = wl.WORKLOADS[1].replace(family=family, n_heads=256 // hd, head_dim=hd, d_ff=d_ff, n_tasks=5,
                                lora_targets=("q", "v", "o", "gate", "up", "down") if family == "decoder"
                                else ("q", "k", "o", "up", "down"))
    log(f"f32 {family} lens={lens} hd={hd} f={d_ff}")
    task = [4, 1, 0, 3, 1][:len(lens)]
    out = _layer_case(w, task, lens, [8, 64, 0, 32, 16])
    _check_layer(w, out[0], out[1], out[2], out[3], range(len(lens)))


@pytest.mark.parametrize("idx,lens", [(2, [1]), (2, [63, 1, 1]), (2, [129, 64]), (2, [511, 512]), (3, [1, 2, 60, 1]),
                                      (3, [300, 64, 256, 400]), (2, [1100, 3, 90]), (3, [700, 40, 333, 1])])
def test_direct_tiles_against_oracle(idx, lens):
    """Encoder layers on the 64- and 128-row tiles, both sides of the
    small-batch threshold, every rank class and a bare task."""
    w = wl.WORKLOADS[idx].replace(n_tasks=4, lora_targets=("q", "k", "v", "o", "up", "down"))
    log(f"direct tiles {w.name} lens={lens}")
    out = _layer_case(w, [3, 0, 2, 3][:len(lens)], lens, [8, 16, 0, 16] if len(lens) < 4 else [8, 16, 64, 32], b_std=0.03)
    _check_layer(w, out[0], out[1], out[2], out[3], range(len(lens)))


def test_operands_of_2_31_elements():
    """1024 rows x 2^21 MLP columns: the down projection's activations need
    64-bit offsets and take the kernel for such operands, with adapters of one
    and two 32-column steps and a bare task."""
    w = wl.WORKLOADS[2].replace(d=64, n_heads=1, d_ff=1 << 21, n_tasks=3, lora_targets=("q", "up", "down"))
    log("operands of 2^31 elements")
    out = _layer_case(w, [2, 0, 1, 2, 0], [1, 9, 500, 4, 510], [16, 0, 40], b_std=0.03)
    pl = out[1]
    _check_layer(w, *out, [p for p in range(5) if pl["cu_seqlens"][p + 1] - pl["cu_seqlens"][p] < 10])


@pytest.mark.parametrize("n", [1, 3, 33, 64, 65, 128, 129])
@pytest.mark.parametrize("max_rank", [8, 32, 64])
def test_decode_rows_same_beside_others(n, max_rank):
    """Decode rows of the split-K path: the same bits alone (the shrink in the
    GEMM's launch) and among n rows of other tasks, either side of 64 and 128
    rows, ranks in each shrink width and a rank-0 task."""
    w = wl.WORKLOADS[5].replace(d=2048, n_heads=16, d_ff=5504, n_tasks=70)
    ranks = np.array([[0, 8, max_rank][t % 3] for t in range(70)], np.int32)
    model = R.Model(w, n_layers=1, ranks=ranks, b_std=0.05)
    r = np.random.default_rng(n)
    task = np.concatenate([[1], r.integers(0, 70, size=n - 1)]).astype(np.int32)
    ctx = np.concatenate([[77], r.integers(0, 200, size=n - 1)]).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(5)
    kv = torch.randn(2, 16, 78, 128, generator=g, device="cuda").to(torch.bfloat16)

    def run(m):
        slots = int((ctx[:m] + 1).sum())
        start = np.concatenate([[0], np.cumsum(ctx[:m] + 1)[:-1]]).astype(np.int32)
        pb = B.Batch(task[:m], np.ones(m, np.int32), 70, ctx_len=ctx[:m], kv_start=start)
        order = np.argsort(task[:m], kind="stable")
        rows = np.concatenate([seeded_rows(1, w.d, 3), seeded_rows(n, w.d, 4)])[:m][order]
        k = torch.randn(16, slots, 128, generator=g, device="cuda").to(torch.bfloat16)
        v = k.clone()
        k[:, :78], v[:, :78] = kv[0], kv[1]
        x = torch.empty(m, w.d, device="cuda")
        set_rows(x, rows)
        ws = torch.empty(B.vfm_workspace_size(model.cfg, pb.c, model.lora_c(0)), dtype=torch.uint8, device="cuda")
        B.vfm_layer_forward(model.cfg, model.c_layers[0], model.lora_c(0), pb.c, x, k, v, slots, ws)
        return x[int(np.nonzero(order == 0)[0][0])].cpu()

    log(f"decode rows n={n} max_rank={max_rank}")
    assert torch.equal(run(1), run(n))


def _decode_layer(w, model, n_tasks, ids, rows, ctx):
    """One decode row of each of tasks ids (ascending) in a table of n_tasks,
    ids[i] with adapter i of the model; returns a callable and its x."""
    ad = model.adapters[0]
    at = {int(t): i for i, t in enumerate(ids)}
    ranks = np.array([int(ad.rank[at[t]]) if t in at else 0 for t in range(n_tasks)], np.int32)
    factors = {p: ([ad.a(p, at[t]) if t in at else None for t in range(n_tasks)],
                   [ad.b(p, at[t]) if t in at else None for t in range(n_tasks)]) for p in ad.A}
    tab = B.LoraTable(n_tasks, ranks, np.full(n_tasks, 2.0), factors, max_rank=ad.max_rank)
    n = len(ids)
    start = (np.arange(n) * (ctx + 1)).astype(np.int32)
    pb = B.Batch(np.asarray(ids, np.int32), np.ones(n, np.int32), n_tasks, ctx_len=np.full(n, ctx, np.int32),
                 kv_start=start)
    slots = n * (ctx + 1)
    g = torch.Generator(device="cuda").manual_seed(5)
    k, v = (torch.randn(w.n_heads, slots, w.head_dim, generator=g, device="cuda").to(w.torch_dtype) for _ in range(2))
    x = torch.empty(n, w.d, device="cuda")
    ws = torch.empty(B.vfm_workspace_size(model.cfg, pb.c, tab.c), dtype=torch.uint8, device="cuda")

    def run():
        B.vfm_layer_forward(model.cfg, model.c_layers[0], tab.c, pb.c, x, k, v, slots, ws)

    set_rows(x, rows)
    return run, x, (tab, pb)


@pytest.mark.parametrize("n_tasks", [64, 65, 129, 4096, 4097, 9001])
def test_decode_rows_same_in_a_larger_table(n_tasks):
    """Decode rows whose split shrink runs in the GEMM's launch find their
    task in tables up to and past what one and two rounds of the search cover:
    the same bits as in a table of five, ids at its ends and beside each other."""
    w = wl.WORKLOADS[5].replace(d=2048, n_heads=16, d_ff=5504, n_tasks=5)
    model = R.Model(w, n_layers=1, ranks=np.array([8, 16, 0, 32, 16], np.int32), b_std=0.05)
    rows = seeded_rows(5, w.d, 3)
    log(f"decode in a table of {n_tasks}")
    ids = [0, n_tasks // 2, n_tasks // 2 + 1, n_tasks - 2, n_tasks - 1]
    small, x0, keep0 = _decode_layer(w, model, 5, range(5), rows, 40)
    large, x1, keep1 = _decode_layer(w, model, n_tasks, ids, rows, 40)
    small()
    large()
    assert x0.isfinite().all() and torch.equal(x0, x1)


def test_decode_time_follows_the_batch():
    """One decode row costs about the same among 8192 tasks as among 64 (a
    scan of the whole table in every shrink item took 2.3 times as long)."""
    w = wl.WORKLOADS[5].replace(d=2048, n_heads=16, d_ff=5504, n_tasks=1)
    model = R.Model(w, n_layers=1, ranks=np.array([8], np.int32), b_std=0.05)
    t = {}
    for n in (64, 8192):
        run, _, keep = _decode_layer(w, model, n, [n // 2], seeded_rows(1, w.d, 3), 100)
        log(f"decode row among {n} tasks")
        t[n] = _us(run)
        log(f"  {t[n]:.1f} us")
    assert t[8192] < 1.6 * t[64], t


def _spread(w, model, n_tasks, n, run_of):
    """Time of a layer over n one-row requests, all of one task or each of its
    own: {distinct tasks: us}; run_of makes the call for task ids."""
    t = {}
    for k in (1, n):
        ids = np.sort(np.arange(n, dtype=np.int32) * (n_tasks // n) if k == n else np.zeros(n, np.int32))
        run, keep = run_of(ids)
        t[k] = _us(run)
        log(f"  {k} tasks {t[k]:.1f} us")
    return t


def test_narrow_decode_time_of_many_tasks():
    """64 decode rows of a 1024-wide decoder at rank 64, each row of a task of
    its own and all of one task: neither much longer than the other (LoRA steps
    one task after another in a tile: 370 against 129 us; the shrink's 16-row
    groups one after another: 110 against 192)."""
    w = wl.WORKLOADS[5].replace(d=1024, n_heads=8, d_ff=1024, n_tasks=128)
    model = R.Model(w, n_layers=1, ranks=np.full(128, 64, np.int32), b_std=0.05)
    log("narrow decode, 64 rows")

    def run_of(ids):
        ctx = np.full(64, 100, np.int32)
        pb = B.Batch(ids, np.ones(64, np.int32), 128, ctx_len=ctx, kv_start=(np.arange(64) * 101).astype(np.int32))
        k, v = (torch.randn(8, 64 * 101, 128, device="cuda").to(w.torch_dtype) for _ in range(2))
        x = torch.randn(64, w.d, device="cuda")
        ws = torch.empty(B.vfm_workspace_size(model.cfg, pb.c, model.lora_c(0)), dtype=torch.uint8, device="cuda")
        return lambda: B.vfm_layer_forward(model.cfg, model.c_layers[0], model.lora_c(0), pb.c, x, k, v, 64 * 101, ws), pb

    t = _spread(w, model, 128, 64, run_of)
    assert t[64] < 2 * t[1] and t[1] < 1.5 * t[64], t


@pytest.mark.parametrize("lens,d,hd,d_ff", [
    ([129], 4096, 128, 11008), ([150, 106], 4096, 128, 11008), ([257], 4096, 128, 11008), ([333], 4096, 128, 11008),
    ([300, 200], 4096, 128, 11008), ([333, 200], 4096, 128, 11008), ([512, 70], 4096, 128, 11008),
    ([900, 123], 4096, 128, 11008), ([200, 57], 2112, 64, 5504), ([400], 2112, 64, 5504), ([450, 250], 2112, 64, 5504),
    ([800, 200], 2112, 64, 5504)])
def test_walked_splits_same_as_split_launch(lens, d, hd, d_ff):
    """From 257 rows on, where a block walks every K split of its tile, a
    request gets the bits that the split launch gives it alone (at most 128
    rows): each tile shape of the walk (128 x 128, 128 / 192 / 256 x 192), row
    and column tiles whole and ragged, and 129 and 256 rows, the edges of the
    split launch's 256-row tile."""
    w = wl.WORKLOADS[4].replace(d=d, n_heads=d // hd, head_dim=hd, d_ff=d_ff, n_tasks=3)
    model = R.Model(w, n_layers=1, ranks=np.asarray([16, 0, 8], np.int32), b_std=0.05)
    log(f"walked splits d={d} lens={lens}")
    alone = _rows_of(w, model, [2], [100], [5])[0]
    whole = _rows_of(w, model, [2] + [0, 1][:len(lens)], [100] + [n - 100 if i == 0 else n for i, n in enumerate(lens)],
                     [5, 6, 7][:len(lens) + 1])[0]
    assert torch.equal(alone, whole)


@pytest.mark.parametrize("idx,d,hd,d_ff", [(3, 1088, 64, 2880), (4, 1344, 64, 1856), (4, 2048, 128, 5504)])
@pytest.mark.parametrize("ranks", [[16, 8, 24, 0, 16], [64, 16, 32, 48, 8]])
def test_finalize_lora_columns(idx, d, hd, d_ff, ranks):
    """The finalize's LoRA difference: every rank, rows of the factors loaded by
    whole waves and by lanes (ranks that do not divide a wave, slots that end
    inside one), a last wave without all of its columns."""
    w = wl.WORKLOADS[idx].replace(d=d, n_heads=d // hd, head_dim=hd, d_ff=d_ff, n_tasks=5,
                                  lora_targets=wl.PROJ if idx == 4 else ("q", "v", "o", "up", "down"))
    lens = [1, 40, 3, 7, 30]
    log(f"finalize columns {w.name} d={d} ranks={ranks}")
    out = _layer_case(w, [4, 2, 0, 3, 1], lens, ranks, b_std=0.05)
    _check_layer(w, out[0], out[1], out[2], out[3], range(len(lens)))
