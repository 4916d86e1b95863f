"""The d = 128 forward's choice of kernel: problems on both sides of the rule give the two kernels' common result."""
import pytest
import torch

from paper_2205_14135_amd import binding, inputs

pytestmark = pytest.mark.gpu


# fewer work items than compute units on the two-group side, and ragged lengths, whose last blocks are mostly padding,
# on the other; (B, H, N) and the layout of the head and row dimensions
@pytest.mark.parametrize("B,H,N,causal,p,choice", [
    (1, 12, 4096, False, 0.0, "fwd_pp_kernel"),
    (1, 24, 2001, False, 0.0, "fwd_pp_kernel"),
    (16, 16, 1024, False, 0.0, "fwd_kernel"),
    (2, 16, 4198, True, 0.0, "fwd_kernel"),
    (6, 16, 1021, True, 0.0, "fwd_kernel"),
    (1, 8, 8192, True, 0.1, "fwd_kernel"),
    (4, 64, 512, True, 0.1, "fwd_pp_kernel"),
])
@pytest.mark.parametrize("heads_inner", [False, True])
def test_both_kernels_agree_on_either_side(B, H, N, causal, p, choice, heads_inner):
    torch.manual_seed(inputs.BASE_SEED + 1700)
    shape = (B, N, H, 128) if heads_inner else (B, H, N, 128)
    q, k, v = (torch.randn(shape, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    if heads_inner:
        q, k, v = (t.transpose(1, 2) for t in (q, k, v))
    assert binding.attn_debug_kernel_choice(binding.make_params(q, 0.1, causal, p))[0] == choice
    out = {}
    try:
        for variant in ("auto", "base", "pp"):
            binding.attn_debug_set_variant(fwd=variant)
            o, lse = torch.empty_like(q), torch.empty(B, H, N, device="cuda")
            binding.attn_fwd(q, k, v, softmax_scale=128 ** -0.5, causal=causal, dropout_p=p, seed=11, out=o, lse=lse)
            out[variant] = (o.float(), lse)
    finally:
        binding.attn_debug_set_variant(fwd="auto")
    same = "pp" if choice == "fwd_pp_kernel" else "base"
    assert torch.equal(out["auto"][0], out[same][0]) and torch.equal(out["auto"][1], out[same][1])
    # both accumulate in fp32 from the same rounded probabilities and round once: half a unit of bf16 each
    big = out["base"][0].abs().clamp_min(2.0 ** -6)
    assert ((out["base"][0] - out["pp"][0]).abs() / big).max() <= 2.0 ** -7
    assert (out["base"][1] - out["pp"][1]).abs().max() <= 1e-5
