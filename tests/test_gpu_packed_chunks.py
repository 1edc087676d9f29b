"""16-bit layers whose input is repacked, around the number of channel chunks that rows and weights are fetched ahead: reductions of
one chunk, two, odd and even numbers of them, against the oracle and bit for bit on integers."""
import pytest

import oracle
from paper_2209_03704_amd import binding as kst
from paper_2209_03704_amd import workloads as wl
from test_gpu_packed import _run
from test_gpu_parity import TOL, check_exact_with_guards, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Cin", [16, 32, 40, 64, 80])
@pytest.mark.parametrize("B,Cout,N,n,P", [(4, 32, 15, 3, 1), (1, 20, 60, 3, 0), (64, 64, 16, 3, 2), (4, 32, 15, 4, 1), (3, 20, 14, 5, 2)])
def test_few_chunks(B, Cout, N, n, P, Cin):
    layer = wl.Layer("chunks", B, Cin, Cout, N, n, "f16", "relu_normal", w_std=0.1)
    x, w, got = _run(layer, P, 3100 + N + Cin)
    e = rel_err(got.cpu().numpy(), oracle.forward(wl.to_f64(x), wl.to_f64(w), P))
    assert e <= TOL["f16"], "rel err %.3e" % e
    check_exact_with_guards(wl.Layer("chunks_int", B, Cin, Cout, N, n, "f16", "integer"), kst.KST_PATH_AUTO, 3200 + N, P=P)
