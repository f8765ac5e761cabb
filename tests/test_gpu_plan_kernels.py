"""Which kernel decodes each code of a plan: a change of it through
LDPC_BLOCK_PATH rebuilds the table and invalidates a captured graph, also where
both kernels keep the code on chip."""
import pytest

from paper_1204_0334_amd import ldpc

from test_gpu_plan import assert_same, make_case, single_code

pytestmark = pytest.mark.gpu

SPREAD = dict(J=3, L=6, p=2000, gamma=3, ebn0_db=2.0)   # on 16 compute units; =onchip: on one
SHORT = dict(J=3, L=6, p=81, gamma=40, ebn0_db=2.0)


@pytest.mark.parametrize("other", ["onchip", "packages"])
def test_a_change_of_path_invalidates_a_captured_graph(other, monkeypatch):
    monkeypatch.delenv("LDPC_BLOCK_PATH", raising=False)
    specs = [SHORT, SPREAD]
    graphs, llrs = make_case(specs, 9300)
    plan = ldpc.Plan(graphs, [c["gamma"] for c in specs], 12, early_stop=True)
    ws, outs = plan.workspace(), plan.outputs()
    plan.capture(llrs, outs, ws)
    plan.replay()
    assert_same(outs, single_code(graphs, llrs, 12, True), "captured")
    monkeypatch.setenv("LDPC_BLOCK_PATH", other)
    assert_same(plan.decode(llrs, outs=outs, ws=ws), single_code(graphs, llrs, 12, True), other)
    with pytest.raises(ldpc.LdpcError) as e:
        plan.replay()
    assert e.value.status == ldpc.EINVAL
    plan.capture(llrs, outs, ws)
    plan.replay()
    assert_same(outs, single_code(graphs, llrs, 12, True), f"captured with {other}")
