"""Kernel names in the profile summaries: the setup kernels live in unnamed namespaces."""
from paper_1410_2153_amd import counters as C


def test_names_inside_unnamed_namespaces():
    assert C._name("asmg::(anonymous namespace)::k_transfer(int, double const*)") == "asmg::k_transfer"
    assert C._name("void asmg::(anonymous namespace)::k_r0<2>(int)") == "asmg::k_r0<2>"
    assert C._name("void asmg::k_sell<0, double, 1>(int, int const*)") == "asmg::k_sell<0, double, 1>"
