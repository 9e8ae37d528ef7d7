"""The value gradients' output: one that is too short, of another type or not
on the GPU is refused before any launch (the kernels write one element per
entry, in the vectors' type), and the Chebyshev backward gives them one in the
vectors' type whatever type the values have."""
import numpy as np
import pytest
import torch

from paper_0910_4836_amd import spmv as S

N_ROWS, N_COLS, NNZ = 6, 9, 8


def jds():
    ptr = np.array([0, 6, 8], np.int32)
    return S.JDS(N_ROWS, N_COLS, torch.arange(N_ROWS, dtype=torch.int32), torch.arange(N_ROWS, dtype=torch.int32),
                 torch.from_numpy(ptr), ptr, torch.zeros(NNZ, dtype=torch.int32), torch.zeros(NNZ, dtype=torch.float64))


@pytest.mark.parametrize("call", [
    lambda g, x, out: S.spmv_grad_vals_jds(jds(), g, x, out),
    lambda g, x, out: S.spmv_grad_vals_jds_sum(jds(), [(1.0, g, x), (2.0, g, x)], out)], ids=["single", "sum"])
def test_mismatches_raise_before_launch(call):
    # CPU tensors: a call that passed the other checks stops at the device check
    g, x = torch.zeros(N_ROWS, dtype=torch.float64), torch.zeros(N_COLS, dtype=torch.float64)
    with pytest.raises(ValueError, match="out is torch.float32 but g and x are torch.float64"):
        call(g, x, torch.zeros(NNZ, dtype=torch.float32))
    with pytest.raises(ValueError, match="out has 7 elements"):
        call(g, x, torch.zeros(NNZ - 1, dtype=torch.float64))
    with pytest.raises(ValueError, match="vectors of 6 and 9 elements"):
        call(g[1:], x, None)
    with pytest.raises(ValueError, match="vectors of 6 and 9 elements"):
        call(g, x.float(), None)
    with pytest.raises(TypeError, match="float64 or float32"):
        call(g.bfloat16(), x.bfloat16(), None)
    with pytest.raises(ValueError, match="must live on the GPU"):
        call(g, x, torch.zeros(NNZ, dtype=torch.float64))


@pytest.mark.gpu
@pytest.mark.parametrize("steps", [1, 2, 7, 20])
def test_chebyshev_gradient_of_narrower_values(steps):
    """FP32 values with FP64 vectors: the checkpointed backward's sums are those
    of the reverse sweep over stored states, call by call in FP64, and its value
    gradient is their rounding to FP32."""
    import synth
    from gpu_common import to_dev
    from paper_0910_4836_amd import autograd as AG
    r, c, v, n, _ = synth.banded_uniform(n=5000, band=300, dtype=np.float64)
    op = AG.SpMVOperator(S.csr_from_coo(n, n, to_dev(r), to_dev(c), to_dev(v.astype(np.float32))))
    vals = op.J.jd_val.clone().requires_grad_(True)
    x = to_dev(synth.uniform_vector(n, synth.rng_for(5, 4))).requires_grad_(True)
    AG.chebyshev_loss(op, vals, x, steps=steps, checkpoint=5).backward()
    ys = AG.cheb_states(op, vals.detach(), x.detach(), steps)
    bar = [torch.zeros_like(ys[0]) for _ in range(steps)] + [2.0 * ys[steps]]
    dvals = torch.empty(op.nnz, dtype=torch.float64, device="cuda")
    for k in range(steps - 1, -1, -1):
        alpha = 2.0 if k else 1.0
        op.rmatvec(vals.detach(), bar[k + 1], bar[k], alpha=alpha, beta=1.0)
        if k:
            S.spmv_axpby(-1.0, bar[k + 1], 1.0, bar[k - 1])
        S.spmv_grad_vals_jds(op.J, bar[k + 1], ys[k], dvals, alpha=alpha, beta=0.0 if k == steps - 1 else 1.0)
    assert vals.grad.dtype == torch.float32 and torch.equal(vals.grad, dvals.float())
    assert x.grad.dtype == torch.float64 and torch.equal(x.grad, bar[0])
