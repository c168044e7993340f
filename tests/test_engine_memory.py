"""Device memory of the CG engines: the fields that a slot is said to hold, and
the memory that a batch takes for them."""
import gc

import numpy as np
import pytest

import synth

FIELD = {"fp64": 192, "fp32": 96, "fp16": 52, "bf16": 52}  # bytes per odd site


def slot_fields(sloppy, mode):
    """b, x, t_e, t_o in FP64; r and p, and t_e and t_o once more where the inner
    precision is another; the FP32 correction; and what switch mode adds."""
    s = FIELD[sloppy]
    if sloppy == "fp64":
        return 6 * 192
    return 4 * 192 + 4 * s + 96 if mode == "reliable" else 7 * 192 + 4 * s


@pytest.mark.parametrize("sloppy,mode", [(s, m) for s in FIELD for m in ("reliable", "switch") if (s, m) != ("fp64", "switch")])
def test_slot_footprint(sloppy, mode):
    from paper_0905_3331_amd import tmq

    dims = (16, 8, 8, 10)
    o = tmq.solver_opts(sloppy=sloppy, mode=mode)
    per = tmq.footprint_bytes(dims, o, 2) - tmq.footprint_bytes(dims, o, 1)
    assert per == slot_fields(sloppy, mode) * (int(np.prod(dims)) // 2)


@pytest.mark.gpu
@pytest.mark.parametrize("sloppy", ["fp64", "fp32", "fp16"])
def test_memory_of_a_batch(sloppy):
    """A batch of 16 takes its slots' fields, within half an FP64 field of the batch
    (50 MB: partial sums, allocation granularity, code of the batched launches)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0905_3331_amd import tmq

    dims, n = (16, 16, 16, 16), 16
    vh = int(np.prod(dims)) // 2
    lat = tmq.Lattice(dims)
    lat.load_gauge(torch.from_numpy(synth.random_gauge(dims, seed=421)).to("cuda"))
    p = tmq.params(0.1632, 0.01, (1.0, 0.0, 0.0, 0.0))
    o = tmq.solver_opts(tol=1e-3, sloppy=sloppy, sloppy_link="fp32" if sloppy == "fp32" else "fp16")
    bs = [torch.ones(vh, 4, 3, dtype=torch.complex128, device="cuda") for _ in range(n)]
    xs = [torch.zeros_like(b) for b in bs]
    lat.solve(p, bs[0], o)  # (code and the engine of one slot, which the batch replaces)
    gc.collect()  # (lattices that other tests left)
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    lat.solve_batch([p] * n, bs, o, xs)
    torch.cuda.synchronize()
    took = free0 - torch.cuda.mem_get_info()[0]
    want = (n - 1) * slot_fields(sloppy, "reliable") * vh
    assert abs(took - want) < n * 192 * vh // 2, (took, want)
    lat.close()


@pytest.mark.gpu
@pytest.mark.parametrize("sloppy", ["fp64", "fp32"])
@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (34, 10, 6, 14)], ids=lambda d: "x".join(map(str, d)))
def test_server_counts_what_an_engine_holds(sloppy, dims):
    """A server's account of an engine: per slot the fields, three arrays of
    partial sums of 4 per block (the second lattice needs 184 blocks, for the
    z-slabs of a lane pair per site) and the scalars."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0905_3331_amd import tmq

    vh = int(np.prod(dims)) // 2
    blocks = {(4, 4, 4, 4): 8, (34, 10, 6, 14): 184}[dims]
    want = 3 * (slot_fields(sloppy, "reliable") * vh + 3 * 4 * blocks * 8 + 7 * 8 + 8 * 4)
    o = tmq.solver_opts(tol=1e-3, sloppy=sloppy, sloppy_link="fp32")
    p = tmq.params(0.1632, 0.01, (1.0, 0.0, 0.0, 0.0))
    U = torch.from_numpy(synth.random_gauge(dims, seed=422)).to("cuda")
    b = torch.ones(vh, 4, 3, dtype=torch.complex128, device="cuda")
    torch.cuda.synchronize()
    with tmq.Server(max_batch=3) as srv:
        lid = srv.add_lattice(dims, U)
        assert srv.wait(srv.submit(lid, p, b, o), timeout=60)[1].status == 0
        st = srv.stats()
    assert st["peak_bytes"] == want, (st["peak_bytes"], want)
