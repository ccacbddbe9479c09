"""GPU parity of the pass that normalises x in front of the multiplication, at the row lengths where its forms meet: less than a
vector, whole and broken vectors, the longest row of each number of vectors per lane, few and many rows, rows at odd addresses."""
import pytest
import torch

from paper_2511_16964_amd import binding, inputs

from parity import assert_close, dev_epilogue, oracle_rows, run_gpu

pytestmark = pytest.mark.gpu

F32, BF16, F16 = torch.float32, torch.bfloat16, torch.float16
V = {F32: 4, BF16: 8, F16: 8}   # elements per 16 bytes


@pytest.mark.parametrize("dtype", [F32, BF16, F16])
@pytest.mark.parametrize("vecs,M", [(0, 9), (0, 1029), (128, 9), (128, 1029), (256, 1029), (512, 70), (512, 1029), (1024, 9), (2048, 9), (4096, 9)])
@pytest.mark.parametrize("off", [-1, 0, 1])
def test_row_lengths_at_the_edges_of_the_forms(dtype, vecs, M, off):
    K = vecs * V[dtype] + off if vecs else V[dtype] + off   # 64 lanes x 2, 4, 8 vectors; a workgroup's x 4, 8, 16
    prob = inputs.random_problem(91, M, 17, K, dtype, ["bias"], ln_pre=True)
    print("[case]", dtype, M, K, flush=True)
    got, call = run_gpu(prob, "auto" if M > 4 else "general", poison=True)
    assert "ln_pre=pass" in call.plan(), call.plan()
    assert_close(got, oracle_rows(prob), dtype, what="%s %d x %d %s" % (dtype, M, K, call.plan()))


@pytest.mark.parametrize("dtype", [F32, BF16, F16])
@pytest.mark.parametrize("M,K", [(1030, 1000), (1030, 1003), (33, 4099), (33, 9000)])
@pytest.mark.parametrize("gamma,beta", [(True, True), (False, True), (True, False)])
def test_rows_and_affine_parts_at_odd_addresses(dtype, M, K, gamma, beta):
    prob = inputs.random_problem(92, M, 40, K, dtype, ["bias", "relu"], ln_pre=True)
    e = prob.epilogue[0]
    prob.epilogue[0] = ("layernorm_pre", e[1] if gamma else None, e[2] if beta else None, e[3])
    odd = lambda t: torch.cat([t.new_zeros(1), t.flatten()]).to("cuda:0")[1:].view(t.shape)
    x = torch.zeros(M, K + 5, dtype=dtype, device="cuda:0")[:, 1:K + 1]
    x.copy_(prob.x.to("cuda:0"))
    ep = dev_epilogue(prob.epilogue)
    ep[0] = ("layernorm_pre", odd(e[1]) if gamma else None, odd(e[2]) if beta else None, e[3])
    print("[case] odd", dtype, M, K, gamma, beta, flush=True)
    call = binding.Call(x, prob.w.to("cuda:0"), prob.b.to("cuda:0"), ep)
    got = call.run().cpu()
    assert "ln_pre=pass" in call.plan(), call.plan()
    assert_close(got, oracle_rows(prob), dtype, what="odd addresses %s" % call.plan())
