"""The big-tile kernels at the edges of their tiles: every count of 32-token blocks with its first and
last row, K stages that do not fill the register ring, a partial last block of output rows, both weight
layouts, and more items than workgroups (so that tiles run in sorted order)."""
import numpy as np
import pytest

from paper_2607_23099_amd import damoe, synth
from tests.gpu_common import TOL, bf16_rows, log, oracle_rows, row_err, tile_rows, torch_cuda

pytestmark = pytest.mark.gpu

# Tokens of each expert: both ends of each block count 1 .. 8, whole tiles with and without a
# remainder, and an empty expert.
EDGES = [1, 32, 33, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 224, 225, 255, 256, 257, 300, 512, 0, 513]


def _routing(counts, seed):
    """k = 1 routing that gives expert e exactly counts[e] tokens, in a random token order."""
    rng = np.random.default_rng(seed)
    ids = np.repeat(np.arange(len(counts)), counts).astype(np.int32)
    rng.shuffle(ids)
    w = rng.uniform(0.5, 1.5, (len(ids), 1)).astype(np.float32)
    return synth.Routing(ids=ids[:, None], w=w, logp=np.zeros(len(counts)), E=len(counts), k=1, alpha=None)


def _variant(name):
    return [damoe.variant_name(v) for v in range(damoe.num_variants())].index(name)


@pytest.mark.parametrize("packed", [False, True], ids=["rowmajor", "packed"])
@pytest.mark.parametrize("wdtype,H,I,names", [
    ("bf16", 384, 128, ["big_bm256"]),          # 6 and 2 stages; GEMM2 rows 256 + 128
    ("bf16", 128, 1920, ["big_bm256"]),         # 2 and 30 stages; 15 feature blocks, more items than CUs
    ("fp8", 512, 1536, ["big_bm256", "big8_bm256", "deep_bm64", "deep8_bm64"]),  # all with this GEMM1
])
def test_big_tile_edges(wdtype, H, I, names, packed):
    torch = torch_cuda()
    from paper_2607_23099_amd.moe import DeviceLayer, Path
    sh = synth.Shape(f"edges-{wdtype}", E=len(EDGES), k=1, H=H, I=I, shape_id=61, wdtype=wdtype)
    r = _routing(EDGES, 5)
    dl = DeviceLayer(sh, packed=packed)
    path = Path(dl, r.T)
    path.set_routing(r)
    path.fill_x(r.T, 3)
    path.route(r.T)
    ref = oracle_rows(sh, r, 3, np.arange(r.T))
    for name in names:
        for rep in range(2):  # the work queues come back to zero
            path.y.fill_(float("nan"))
            path.fused(r.T, _variant(name))
            torch.cuda.synchronize()
            err = row_err(bf16_rows(path.y, np.arange(r.T)), ref)
            log(f"{name} {wdtype} H={H} I={I} packed={packed}: {err:.4f}")
            # the layer's bound of its weight type: h, out and y rounded to bf16 (and h to e4m3)
            assert err <= TOL[wdtype], (name, err)
    assert damoe.read_device_error(path.ws) == 0


@pytest.mark.parametrize("wdtype", ["bf16", "fp8"])
def test_row_major_weights_keep_up(wdtype):
    """A few tokens on each of 48 experts: the layer call on row-major weights against packed ones.  Gathered
    into LDS they take 1.4-1.7 times as long; loaded straight into MFMA operands it was 2.6-3.4 times."""
    torch = torch_cuda()
    from paper_2607_23099_amd.moe import DeviceLayer, Path
    sh = synth.Shape(f"rows-{wdtype}", E=48, k=8, H=7168, I=2048, shape_id=63, wdtype=wdtype)
    T = 64
    r = synth.routing(sh.E, sh.k, T, 10.0, [64])
    times = []
    for packed in (True, False):
        path = Path(DeviceLayer(sh, packed=packed), T)
        path.set_routing(r)
        path.fill_x(T, 5)
        path.route(T)
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(10)]
        path.fused(T, _variant("big_bm256"))
        for a, b in zip(ev[::2], ev[1::2]):
            a.record()
            path.fused(T, _variant("big_bm256"))
            b.record()
        torch.cuda.synchronize()
        times.append(np.median([a.elapsed_time(b) for a, b in zip(ev[::2], ev[1::2])]))
        assert damoe.read_device_error(path.ws) == 0
        del path
    log(f"{wdtype} T={T}: packed {times[0]:.3f} ms, row-major {times[1]:.3f} ms")
    assert times[1] <= 2.1 * times[0]


def test_more_tiles_than_a_sorted_launch_takes():
    """A list of more than 8192 tiles of 256 rows: GEMM1 runs it in list order over many items a workgroup."""
    torch = torch_cuda()
    from paper_2607_23099_amd.moe import DeviceLayer, Path
    sh = synth.Shape("many-tiles", E=18, k=16, H=128, I=256, shape_id=62)
    T = 131400
    rng = np.random.default_rng(9)
    ids = rng.random((T, sh.E)).argsort(axis=1)[:, : sh.k].astype(np.int32)
    w = rng.uniform(0.02, 0.1, (T, sh.k)).astype(np.float32)
    r = synth.Routing(ids=ids, w=w, logp=np.zeros(sh.E), E=sh.E, k=sh.k, alpha=None)
    path = Path(DeviceLayer(sh), T)
    path.set_routing(r)
    path.fill_x(T, 4)
    path.route(T)
    assert len(path.tiles(T, 4)) > 8192
    rows = tile_rows(r, sh.E, n_min=128, seed=2)
    ref = oracle_rows(sh, r, 4, rows)
    for _ in range(2):
        path.y.fill_(float("nan"))
        path.fused(T, _variant("big_bm256"))
        torch.cuda.synchronize()
        err = row_err(bf16_rows(path.y, rows), ref)
        log(f"{len(path.tiles(T, 4))} tiles: {err:.4f}")
        assert err <= TOL["bf16"]
        assert bool(torch.isfinite(path.y[:T].float()).all())
    assert damoe.read_device_error(path.ws) == 0
