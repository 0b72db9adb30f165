"""bench.py's parity check: it judges the launch it makes whatever else is queued on the default stream, and a failed
check shows in the exit status."""
from types import SimpleNamespace

import pytest
import torch

import bench


def test_failed_parity_is_an_exit_status():
    ok, bad = {"parity": {"pass": True}}, {"parity": {"pass": False}}
    assert bench.exit_code(ok) == 0 and bench.exit_code({"parity": None}) == 0
    assert bench.exit_code(bad) == bench.PARITY_EXIT != 0
    assert bench.exit_code({**ok, "prefill_extra": {"parity_pass": True}}) == 0
    assert bench.exit_code({**ok, "prefill_extra": {"parity_pass": False}}) == bench.PARITY_EXIT


# The check poisons the outputs and calls the product on a side stream.  With milliseconds of work queued on the default
# stream, a poisoning fill there lands after the product's stores unless the two are ordered.
@pytest.mark.gpu
@pytest.mark.parametrize("M", [1, 8])
def test_parity_check_does_not_depend_on_the_default_stream(M, monkeypatch):
    print("case: bench parity beside a busy default stream", M, flush=True)
    import paper_2502_11880_amd as B
    from oracle import bitnet_oracle as O
    from paper_2502_11880_amd import inputs
    from tests import hip_runner as H

    N, K, layout, args = 1024, 1536, "i2s", SimpleNamespace(workload=0)
    packed, scale = H.pack(inputs.weight_f32(N, K, seed=inputs.seed_for(0, 0)), layout)
    x = inputs.activation_f32(M, K, seed=5).to(H.DEV)
    y = torch.empty((M, N), dtype=torch.float32, device=H.DEV)
    fargs = [[[B.FusedArgs([packed], [scale], [y])]]]
    busy = torch.empty(1 << 30, dtype=torch.uint8, device=H.DEV)
    ws = H.workspace(layout, M, N, K)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    epilogue = O.epilogue

    def epilogue_then_busy(*a):                       # the oracle's last step before the check's launches
        r = epilogue(*a)
        for i in range(20):
            busy.fill_(i)                             # about 0.2 ms each
        return r

    def check():
        return bench.parity_check(args, layout, M, [("p", K, N)], [["p"]], {"p": (K, N)}, [x], {"p": y}, fargs, 1, ws,
                                  stream)

    assert check()["pass"]                            # loads every kernel, so that the next pass does not wait for that
    monkeypatch.setattr(O, "epilogue", epilogue_then_busy)
    result = check()
    assert result["pass"], result
