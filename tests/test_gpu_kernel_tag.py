"""qed_info names the kernel that runs."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_in,mode,prec,var,tag", [
    (3, 1, "sum", "fp64", {}, "nin1_nout3_p0_m0_coop_l8_b64"),
    (4, 1, "sum", "fp64", dict(rewrite=1), "nin1_nout4_p0_m0_coop_l32_b64_d1"),
    (5, 1, "per_point", "fp64", {}, "nin1_nout5_p0_m1_pair_l2_b256"),
    (1, 6, "per_point", "fp64", dict(rewrite=1), "nin6_nout1_p0_m1_pair_l2_b64_d1"),
    (3, 1, "sum", "fp64", dict(lane_bits=7), "nin1_nout3_p0_m0_e56_l7_o0_b256_s2_j1_r0_w0"),
    (5, 1, "per_point", "fp32c", {}, "nin1_nout5_p1_m1_e0_l0_o0_b256_s3_j1_r520_w0_f1")])
def test_kernel_tag(n, n_in, mode, prec, var, tag):
    from paper_2511_19456_amd.qedx import QedProcess, make_variant
    info = QedProcess(n, mode, prec, make_variant(**var) if var else None, n_in=n_in).info()
    assert info["kernel_tag"] == tag
    if "_pair_" in tag or "_coop_" in tag:
        assert f"_l{info['lanes_per_point']}_b{info['block']}" in tag
