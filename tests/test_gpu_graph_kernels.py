"""FP64 processes with a given kernel shape: the kernels that follow the graph
node by node, with and without the distributive rewrite, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import qed_oracle as O
from paper_2511_19456_amd import inputs
from parity import REL_FP64, check_fp64, per_point_ref

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("n_in,n,mode,rewrite,N", [
    (1, 1, "sum", 0, 333), (1, 2, "sum", 0, 333), (1, 3, "sum", 0, 517), (1, 4, "sum", 0, 97), (3, 1, "sum", 0, 389),
    (1, 2, "sum", 1, 333), (1, 3, "sum", 1, 517), (1, 4, "sum", 1, 97),
    (1, 3, "per_point", 0, 601), (1, 4, "per_point", 0, 300), (1, 5, "per_point", 0, 200), (1, 6, "per_point", 0, 40),
    (1, 4, "per_point", 1, 300), (1, 5, "per_point", 1, 200), (1, 6, "per_point", 1, 40), (6, 1, "per_point", 1, 40)])
def test_graph_kernels_fp64(n_in, n, mode, rewrite, N):
    from paper_2511_19456_amd.qedx import QedProcess, make_variant
    if n_in == 1:
        u, hel = inputs.rambo_inputs(35, n, N, with_helicities=True)
        mom = O.momenta_soa_from_uniforms(u, 6.0 + 3 * n, n).numpy()
    else:
        mom, hel = inputs.crossed_inputs(35 + n_in, n_in, N, with_helicities=True)
    p = QedProcess(n, mode, "fp64", make_variant(block=256, rewrite=rewrite), n_in=n_in)
    tag = p.info()["kernel_tag"]
    assert "_b256_" in tag and tag.endswith("_d1") == bool(rewrite)
    md = torch.as_tensor(mom, device=DEV)
    if mode == "sum":
        ref = O.m2(mom, n, "sum", n_in=n_in).numpy()
        assert np.abs(p.eval(md).cpu().numpy() / ref - 1.0).max() < REL_FP64
    else:
        got = p.eval(md, torch.as_tensor(hel.astype(np.int32), device=DEV)).cpu().numpy()
        ref, kap = per_point_ref(mom, n, hel, n_in=n_in)
        check_fp64(got, ref, kap, f"{n_in} -> {n}")


@pytest.mark.parametrize("N", [517, 773, 1])
def test_matrix_core_joins_against_the_same_graphs_vector_joins(N):
    """The matrix cores sum a join's products in another order only."""
    from paper_2511_19456_amd.qedx import QedProcess, make_variant
    u, _ = inputs.rambo_inputs(33, 3, N)
    m = torch.as_tensor(O.momenta_soa_from_uniforms(u, 10.0, 3).numpy(), device=DEV)
    mat = QedProcess(3, "sum", "fp64", make_variant(rewrite=1, order=128))
    vec = QedProcess(3, "sum", "fp64", make_variant(rewrite=1, block=256))
    assert mat.info()["kernel_name"].endswith("_mfma") and "_l5_o0_b256_" in vec.info()["kernel_tag"]
    assert (mat.eval(m) / vec.eval(m) - 1.0).abs().max().item() < 1e-13
