"""Operator applications recorded into a HIP graph.  A program applies an
operator once (which tunes it and makes its work fields) and may then capture
any call of that operator and precision (a lattice keeps the work fields of the
precision it applied last): in place or not, whatever the boundary phases.
Replays are compared with eager calls of another lattice handle."""
import numpy as np
import pytest

import synth
from test_gpu_parity import THETA, THETA_GEN, dev, tmq  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def capture(call):
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        call()
    return g


# below and above the sizes where the half-sweeps read canonical buffers and
# where a 16-bit field leaves the split kernel
@pytest.mark.parametrize("dims", [(8, 8, 8, 8), (32, 16, 14, 16)], ids=lambda d: "x".join(map(str, d)))
def test_captured_after_one_call(tmq, dims):  # noqa: F811
    U = dev(synth.random_gauge((4, 4, 2, 4), seed=431))
    U = U.repeat(*(d // u for d, u in zip(dims, U.shape[:4])), 1, 1, 1).contiguous()
    V = int(np.prod(dims))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(81)
    full = torch.view_as_complex(torch.randn(V, 4, 3, 2, dtype=torch.float64, device="cuda", generator=gen))
    src = full[: V // 2].contiguous()
    lat, other = tmq.Lattice(dims), tmq.Lattice(dims)
    lat.load_gauge(U)
    other.load_gauge(U)
    pt, pg = tmq.params(0.1632, 0.004, THETA), tmq.params(0.1632, 0.004, THETA_GEN)
    out, fout, buf, fbuf = torch.empty_like(src), torch.empty_like(full), src.clone(), full.clone()
    for p in (pt, pg):
        # per case: the one call, the result, the work buffer and what goes into it, the captured call
        cases = [(lambda: lat.apply_Q_full(pt, +1, full, out=fout), other.apply_Q_full(p, +1, full), full, fbuf,
                  lambda: lat.apply_Q_full(p, +1, fbuf, out=fbuf))]
        for prec in ("fp64", "fp32", "fp16", "bf16"):
            cases.append((lambda prec=prec: lat.apply_Qhat(pt, +1, src, out=out, prec=prec),
                          other.apply_Qhat(p, +1, src, prec=prec), src, buf,
                          lambda prec=prec: lat.apply_Qhat(p, +1, buf, out=buf, prec=prec)))
        # Qhat in FP64 has the work fields of Qhat^+ Qhat^- too
        cases.append((lambda: lat.apply_QhatQhat(pt, src, out=out), other.apply_Qhat(p, +1, src), src, buf,
                      lambda: lat.apply_Qhat(p, +1, buf, out=buf)))
        for n, (once, want, given, work, call) in enumerate(cases):
            once()
            torch.cuda.synchronize()
            g = capture(call)
            for _ in range(3):
                work.copy_(given)
                g.replay()
                torch.cuda.synchronize()
                assert torch.equal(work, want), n
            del g
    lat.close()
    other.close()
