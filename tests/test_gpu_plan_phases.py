"""A plan whose last codes run in launches of their own after codes of the phase
launches (rows of weight 12, which no other kernel takes): the threads that fill
up a phase launch's last block leave their results alone."""
import pytest
import torch

from paper_1204_0334_amd import ldpc

from test_gpu_plan import assert_same, make_case, single_code

pytestmark = pytest.mark.gpu

PHASES = dict(J=3, L=12, p=230, gamma=33, ebn0_db=3.0)   # 8280 edges: too many for a frame's packages in LDS
ONCHIP = dict(J=3, L=6, p=81, gamma=100, ebn0_db=2.0)
SMALL = dict(J=3, L=18, p=36, gamma=33, ebn0_db=3.5)


@pytest.mark.parametrize("specs", [[PHASES, ONCHIP], [ONCHIP, PHASES, SMALL], [PHASES, ONCHIP, PHASES, SMALL]])
@pytest.mark.parametrize("early", [True, False])
def test_codes_of_one_launch_after_phase_codes(specs, early, monkeypatch):
    monkeypatch.delenv("LDPC_BLOCK_PATH", raising=False)
    graphs, llrs = make_case(specs, 9100)
    plan = ldpc.Plan(graphs, [c["gamma"] for c in specs], 20, early_stop=early)
    ws, outs = plan.workspace(), plan.outputs()
    refs = single_code(graphs, llrs, 20, early)
    for rep in range(4):
        for o in outs:
            for t in o:
                t.zero_()
        torch.cuda.synchronize()
        ldpc.timing_read()
        ldpc.timing_enable(True)
        plan.decode(llrs, outs=outs, ws=ws)
        torch.cuda.synchronize()
        ldpc.timing_enable(False)
        t = ldpc.timing_read()
        assert t["plan_check_node"][0] > 0 and t["onchip_decode"][0] == len([c for c in specs if c is not PHASES])
        assert_same(outs, refs, f"codes of one launch after phase codes, {rep}")
