"""A plan whose last codes run on chip after codes of the phase launches: the
threads that fill up a phase launch's last block leave their results alone."""
import pytest
import torch

from paper_1204_0334_amd import ldpc

from test_gpu_plan import assert_same, make_case, single_code

pytestmark = pytest.mark.gpu

PACKAGES = dict(J=3, L=18, p=36, gamma=33, ebn0_db=3.5)
ONCHIP = dict(J=3, L=6, p=81, gamma=100, ebn0_db=2.0)


@pytest.mark.parametrize("specs", [[PACKAGES, ONCHIP], [ONCHIP, PACKAGES, ONCHIP], [PACKAGES, ONCHIP, PACKAGES]])
@pytest.mark.parametrize("early", [True, False])
def test_on_chip_codes_after_phase_codes(specs, early, monkeypatch):
    monkeypatch.delenv("LDPC_BLOCK_PATH", raising=False)
    graphs, llrs = make_case(specs, 9000)
    plan = ldpc.Plan(graphs, [c["gamma"] for c in specs], 20, early_stop=early)
    ws, outs = plan.workspace(), plan.outputs()
    refs = single_code(graphs, llrs, 20, early)
    for _ in range(5):
        for o in outs:
            for t in o:
                t.zero_()
        plan.decode(llrs, outs=outs, ws=ws)
        assert_same(outs, refs, "on-chip codes after phase codes")


def test_a_plan_created_for_the_phase_launches(monkeypatch):
    # its workspace serves the other decoders too: a frame on several compute
    # units (whose words lie in the code's region) and on one
    long = dict(J=3, L=18, p=1700, gamma=16, ebn0_db=3.5)
    monkeypatch.setenv("LDPC_BLOCK_PATH", "packages")
    graphs, llrs = make_case([ONCHIP, long], 9100)
    plan = ldpc.Plan(graphs, [ONCHIP["gamma"], long["gamma"]], 15, early_stop=True)
    ws = plan.workspace()
    assert_same(plan.decode(llrs, ws=ws), single_code(graphs, llrs, 15, True), "created and run for the phase launches")
    monkeypatch.delenv("LDPC_BLOCK_PATH")
    assert_same(plan.decode(llrs, ws=ws), single_code(graphs, llrs, 15, True), "run as ldpc_decode does")
