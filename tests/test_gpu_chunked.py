"""GPU parity of the token-chunked two-stream schedule: per-token outputs are bit-identical to the
unchunked schedule (a row's GEMM results do not depend on its tile mates), weight gradients match
the CPU oracle within the bf16 tolerance."""
import numpy as np
import pytest
import torch

from paper_2605_11005_amd import workloads as W
from paper_2605_11005_amd.chunked import ChunkedLayer
from paper_2605_11005_amd.layer import upload
from tests.gpu_util import TOL, gpu_layer, host, make_inputs, oracle_layer, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_chunks", [2, 4, 8])     # chunks of 512 tokens take the kernel for few rows, the whole batch does not
def test_chunked_schedule_matches_unchunked_and_oracle(n_chunks):
    wl = W.DSV3.scaled(name="dsv3-chunked", T=4096, d=512, f=256)
    print(f"case {wl.name} chunks={n_chunks}", flush=True)
    inp = make_inputs(wl)
    fw, bw = oracle_layer(wl, inp)
    dev, ref = gpu_layer(wl, inp)
    ch = ChunkedLayer(wl, n_chunks)
    for b in ch.bufs:
        for name in ("y", "dx", "d_o", "dxp"):
            getattr(b, name).fill_(5.0)
    ch.bufs[0].dw1.fill_(5.0); ch.bufs[0].dw3.fill_(5.0); ch.bufs[0].dw2.fill_(5.0)
    for _ in range(2):                      # twice: the second pass must not depend on the first
        ch.forward(dev)
        ch.backward(dev)
    torch.cuda.synchronize()
    assert torch.equal(ch.y(), ref.y), "y must be bit-identical to the unchunked schedule"
    assert torch.equal(ch.dx(), ref.dx), "dx must be bit-identical to the unchunked schedule"
    assert rel_err(host(ch.y()), fw["y"]) < TOL["bf16"]
    for name, got, want in (("dw1", ch.bufs[0].dw1, bw["dw1"]), ("dw3", ch.bufs[0].dw3, bw["dw3"]),
                            ("dw2", ch.bufs[0].dw2, bw["dw2"])):
        g = host(got)
        for e in range(wl.e_cnt):
            if fw["counts"][e] == 0:
                assert not g[e].any()
            else:
                assert rel_err(g[e], want[e]) < TOL["bf16"], (name, e)
    counts = sum(host(b.counts) for b in ch.bufs)
    assert (counts == fw["counts"]).all()
