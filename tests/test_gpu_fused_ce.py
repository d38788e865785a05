"""GPU parity of the fused in-place cross-entropy against the fp64 oracle on the same bf16 logits.

Tolerances: the loss is an fp32 reduction over up to 128K terms: |loss - oracle| <= 2e-4 (relative error of the
exponentials ~1e-6, of the logarithm likewise; the logits themselves are exact).  The gradient is rounded to bf16:
|g - oracle| <= 2^-8 |oracle| + 2^-8 |grad_scale| * 1e-3 (half an ulp would be 2^-9; the absolute term covers
probabilities whose exponentials carry the fp32 error of the row's log-sum-exp)."""
import numpy as np
import pytest
import torch

from oracle import fused_ce_oracle as orc

pytestmark = pytest.mark.gpu

CASES = [  # rows, vocab, row stride, spread of the logits
    (5, 8, 8, 2.0), (33, 4096, 4096, 3.0), (70, 128256, 128256, 2.0), (16, 131072, 131072, 6.0),
    (9, 32000, 32768, 4.0), (3, 151936, 151936, 2.0), (2, 262144, 262144, 1.0), (600, 1024, 1024, 8.0),
]


@pytest.mark.parametrize("rows,vocab,stride,spread", CASES)
def test_parity(rows, vocab, stride, spread):
    from paper_2509_21275_amd.fused_ce import fused_ce_inplace
    g = torch.Generator(device="cpu").manual_seed(1000 + rows + vocab)
    buf = (torch.randn((rows, stride), generator=g) * spread).to(torch.bfloat16)
    targets = torch.randint(0, vocab, (rows,), generator=g, dtype=torch.int32)
    if rows > 2:
        targets[1] = -100                           # an ignored row
        targets[2] = vocab - 1
    # make one row sharply peaked on its target and one peaked elsewhere
    buf[0, int(targets[0])] = 40.0
    if rows > 4:
        buf[4, (int(targets[4]) + 1) % vocab] = 30.0
    scale = 1.0 / rows
    want_loss, want_grad = orc.cross_entropy(buf[:, :vocab].double().numpy(), targets.numpy(), scale)
    dev_buf = buf.cuda()
    pad_before = dev_buf[:, vocab:].clone()
    loss = torch.full((rows,), float("nan"), device="cuda")
    fused_ce_inplace(dev_buf[:, :vocab], targets.cuda(), loss, scale)
    torch.cuda.synchronize()
    got_loss = loss.cpu().double().numpy()
    got_grad = dev_buf[:, :vocab].cpu().double().numpy()
    assert np.all(np.isfinite(got_loss)) and np.all(np.isfinite(got_grad))
    assert np.abs(got_loss - want_loss).max() <= 2e-4 * max(1.0, np.abs(want_loss).max())
    tol = 2.0 ** -8 * np.abs(want_grad) + 2.0 ** -8 * scale * 1e-3
    assert np.all(np.abs(got_grad - want_grad) <= tol), float((np.abs(got_grad - want_grad) - tol).max())
    assert torch.equal(dev_buf[:, vocab:], pad_before)        # the padding of a strided row is not touched
    if rows > 2:
        assert got_loss[1] == 0 and np.all(got_grad[1] == 0)  # ignored row


def test_empty_and_bad_arguments():
    import paper_2509_21275_amd as ca
    from paper_2509_21275_amd.fused_ce import fused_ce_inplace
    z = torch.zeros((0, 64), dtype=torch.bfloat16, device="cuda")
    fused_ce_inplace(z, torch.zeros((0,), dtype=torch.int32, device="cuda"), torch.zeros((0,), device="cuda"))
    z = torch.zeros((2, 12), dtype=torch.bfloat16, device="cuda")     # vocabulary not a multiple of 8
    with pytest.raises(ca.ChunkAttnError):
        fused_ce_inplace(z, torch.zeros((2,), dtype=torch.int32, device="cuda"), torch.zeros((2,), device="cuda"))


@pytest.mark.parametrize("vocab", [32768, 32776, 65536, 65544, 131072, 131080, 135168, 163840, 163848, 188416, 188424, 192512, 262136])
def test_edges_of_the_register_and_lds_variants(vocab):
    """Vocabularies at which the rows' last chunks change place (registers of one variant or the next, LDS, a thread's
    last chunk partly or wholly absent); masked entries (-inf) and, in one row, whole threads of them.  Same tolerances."""
    from paper_2509_21275_amd.fused_ce import fused_ce_inplace
    g = torch.Generator(device="cpu").manual_seed(vocab)
    rows, scale = 4, 0.25
    buf = (torch.randn((rows, vocab), generator=g) * 2.0).to(torch.bfloat16)
    targets = torch.tensor([0, vocab - 1, vocab // 2, 5], dtype=torch.int32)
    buf[1, : vocab // 3] = float("-inf")
    buf[2, vocab // 2 + 8:] = float("-inf")
    buf[3, :] = float("-inf")
    buf[3, 5] = 1.5                                 # one finite logit: loss 0, gradient 0
    want_loss, want_grad = orc.cross_entropy(buf.double().numpy(), targets.numpy(), scale)
    dev, loss = buf.cuda(), torch.full((rows,), float("nan"), device="cuda")
    fused_ce_inplace(dev, targets.cuda(), loss, scale)
    torch.cuda.synchronize()
    got = dev.cpu().double().numpy()
    assert np.abs(loss.cpu().double().numpy() - want_loss).max() <= 2e-4 * max(1.0, np.abs(want_loss).max())
    assert np.all(np.abs(got - want_grad) <= 2.0 ** -8 * np.abs(want_grad) + 2.0 ** -8 * scale * 1e-3)


@pytest.mark.parametrize("vocab", [4096, 131072, 131080, 163840, 163848, 262136])
def test_a_nan_logit_is_not_lost(vocab):
    """A NaN makes its row's loss and gradient NaN, also where every other logit of the threads around it is -inf (their maximum
    is then -inf, and the sum that holds the NaN must not be taken for empty); the other rows are as without it."""
    from paper_2509_21275_amd.fused_ce import fused_ce_inplace
    g = torch.Generator(device="cpu").manual_seed(vocab + 1)
    rows = 5
    buf = (torch.randn((rows, vocab), generator=g) * 2.0).to(torch.bfloat16)
    targets = torch.full((rows,), 8, dtype=torch.int32)
    buf[1, 17] = float("nan")                       # among finite logits
    buf[2, 16:] = float("-inf")                     # the only finite logits are the first two chunks' ...
    buf[2, vocab - 3] = float("nan")                # ... the NaN is in the last chunk
    buf[3, 16:] = float("-inf")
    keep = [0, 3, 4]
    want_loss, want_grad = orc.cross_entropy(buf[keep].double().numpy(), targets[keep].numpy(), 0.5)
    dev, loss = buf.cuda(), torch.zeros((rows,), device="cuda")
    fused_ce_inplace(dev, targets.cuda(), loss, 0.5)
    torch.cuda.synchronize()
    got_loss, got = loss.cpu().double().numpy(), dev.cpu().double().numpy()
    assert np.isnan(got_loss[[1, 2]]).all() and np.isnan(got[1]).all() and np.isnan(got[2]).all()
    assert np.abs(got_loss[keep] - want_loss).max() <= 2e-4 * max(1.0, np.abs(want_loss).max())
    assert np.all(np.abs(got[keep] - want_grad) <= 2.0 ** -8 * np.abs(want_grad) + 2.0 ** -8 * 0.5 * 1e-3)


@pytest.mark.parametrize("rows,vocab", [(1100, 131080), (1100, 163848), (600, 262136), (1100, 4096)])
def test_workgroups_that_run_several_rows(rows, vocab):
    """More rows than workgroups (512): a workgroup's next row refills its registers and LDS and reuses its partial results,
    twice where there are more than 1024 rows.  Maxima and targets differ from row to row; rows around the multiples of 512
    and a few others against the oracle, all losses against PyTorch in float64."""
    from paper_2509_21275_amd.fused_ce import fused_ce_inplace
    g = torch.Generator(device="cuda").manual_seed(rows + vocab)
    buf = torch.randn((rows, vocab), generator=g, device="cuda", dtype=torch.bfloat16)
    buf += torch.linspace(-30.0, 30.0, rows, device="cuda").to(torch.bfloat16)[torch.randperm(rows, generator=g, device="cuda")].view(-1, 1)
    targets = torch.randint(0, vocab, (rows,), generator=g, device="cuda", dtype=torch.int32)
    targets[torch.arange(7, rows, 97, device="cuda")] = -1
    check = [r for r in (0, 1, 7, 255, 510, 511, 512, 513, 1022, 1023, 1024, 1025, rows - 2, rows - 1) if r < rows]
    kept = buf[check].cpu().double().numpy()
    want_all = torch.empty(rows, dtype=torch.float64, device="cuda")
    for r0 in range(0, rows, 64):
        z = buf[r0:r0 + 64].double()
        y = targets[r0:r0 + 64].long()
        want_all[r0:r0 + 64] = torch.where(y < 0, torch.zeros((), dtype=torch.float64, device="cuda"),
                                           torch.logsumexp(z, 1) - z.gather(1, y.clamp(min=0).view(-1, 1)).view(-1))
    loss = torch.full((rows,), float("nan"), device="cuda")
    fused_ce_inplace(buf, targets, loss, 0.5)
    torch.cuda.synchronize()
    assert float((loss.double() - want_all).abs().max()) <= 2e-4 * max(1.0, float(want_all.abs().max()))
    want_loss, want_grad = orc.cross_entropy(kept, targets[check].cpu().numpy(), 0.5)
    got = buf[check].cpu().double().numpy()
    assert np.abs(loss[check].cpu().double().numpy() - want_loss).max() <= 2e-4 * max(1.0, np.abs(want_loss).max())
    assert np.all(np.abs(got - want_grad) <= 2.0 ** -8 * np.abs(want_grad) + 2.0 ** -8 * 0.5 * 1e-3)


@pytest.mark.parametrize("rows,vocab", [
    (511, 65544), (512, 65544), (700, 131064), (520, 131072),            # up to 131072 logits: which kernel depends on the number of rows
    (520, 131080), (515, 163840), (515, 163848), (510, 188424),          # logits that the last-level cache holds ...
    (1300, 131072), (1110, 151936), (900, 188432), (35800, 4096), (2600, 65528)])  # ... and some more than it does
@pytest.mark.parametrize("whole_lines", [False, True])
def test_a_row_and_the_next_one_of_its_workgroup(rows, vocab, whole_lines):
    """A workgroup loads its next row as it stores the one before: rows of a stride that is a multiple of a cache line, or not, some masked (-inf) up to their last
    chunks, around the multiples of 256 and 512 and at the end against the oracle, with the tolerances above; what lies between the rows stays as it was."""
    from paper_2509_21275_amd.fused_ce import fused_ce_inplace
    g = torch.Generator(device="cuda").manual_seed(rows + vocab)
    stride = vocab + 8 if (vocab + 8) % 64 != 0 else vocab + 16
    buf = torch.randn((rows, (vocab + 64) // 64 * 64 if whole_lines else stride), generator=g, device="cuda", dtype=torch.bfloat16)
    buf += torch.linspace(-30.0, 30.0, rows, device="cuda").to(torch.bfloat16)[torch.randperm(rows, generator=g, device="cuda")].view(-1, 1)
    buf[1::5, vocab - vocab // 3:vocab] = float("-inf")
    buf[2::5, 8:vocab // 2] = float("-inf")
    targets = torch.randint(0, 8, (rows,), generator=g, device="cuda", dtype=torch.int32)
    targets[3::5] = vocab - 1
    targets[torch.arange(7, rows, 97, device="cuda")] = -1
    check = [r for r in (0, 1, 2, 3, 7, 254, 255, 256, 257, 258, 511, 512, 513, 767, 768, 1024, rows - 2, rows - 1) if r < rows]
    want_loss, want_grad = orc.cross_entropy(buf[check, :vocab].cpu().double().numpy(), targets[check].cpu().numpy(), 0.5)
    between, loss = buf[:, vocab:].clone(), torch.full((rows,), float("nan"), device="cuda")
    fused_ce_inplace(buf[:, :vocab], targets, loss, 0.5)
    torch.cuda.synchronize()
    got = buf[check, :vocab].cpu().double().numpy()
    assert bool(torch.isfinite(loss).all()) and torch.equal(buf[:, vocab:], between)
    assert np.abs(loss[check].cpu().double().numpy() - want_loss).max() <= 2e-4 * max(1.0, np.abs(want_loss).max())
    assert np.all(np.abs(got - want_grad) <= 2.0 ** -8 * np.abs(want_grad) + 2.0 ** -8 * 0.5 * 1e-3)


@pytest.mark.parametrize("rows,vocab", [
    (1380, 100000), (1060, 131072), (1100, 128256), (900, 151936), (530, 262136),   # a little more than the last-level cache holds
    (16400, 65544), (8200, 131072), (8250, 131064)])                                # more than 2 GiB: several rows to a workgroup of either kernel
@pytest.mark.parametrize("whole_lines", [False, True])
def test_more_than_the_cache_and_more_than_2_gib(rows, vocab, whole_lines):
    """Logits of sizes at which the choice of kernel and of streaming changes, as above: some rows, the last among them, against the oracle; what lies between
    the rows stays as it was."""
    from paper_2509_21275_amd.fused_ce import fused_ce_inplace
    g = torch.Generator(device="cuda").manual_seed(rows + vocab)
    stride = vocab + 8 if (vocab + 8) % 64 != 0 else vocab + 16
    buf = torch.empty((rows, (vocab + 64) // 64 * 64 if whole_lines else stride), device="cuda", dtype=torch.bfloat16)
    for r in range(0, rows, 1024):
        buf[r:r + 1024].normal_(generator=g)
    buf[1::5, vocab - vocab // 3:vocab] = float("-inf")
    targets = torch.randint(0, 8, (rows,), generator=g, device="cuda", dtype=torch.int32)
    targets[3::5] = vocab - 1
    targets[torch.arange(7, rows, 97, device="cuda")] = -1
    check = [r for r in (0, 1, 3, 7, 255, 256, 511, 512, rows // 2, rows - 2, rows - 1)]
    want_loss, want_grad = orc.cross_entropy(buf[check, :vocab].cpu().double().numpy(), targets[check].cpu().numpy(), 0.5)
    between, loss = buf[:, vocab:].clone(), torch.full((rows,), float("nan"), device="cuda")
    fused_ce_inplace(buf[:, :vocab], targets, loss, 0.5)
    torch.cuda.synchronize()
    got = buf[check, :vocab].cpu().double().numpy()
    assert bool(torch.isfinite(loss).all()) and torch.equal(buf[:, vocab:], between)
    assert np.abs(loss[check].cpu().double().numpy() - want_loss).max() <= 2e-4 * max(1.0, np.abs(want_loss).max())
    assert np.all(np.abs(got - want_grad) <= 2.0 ** -8 * np.abs(want_grad) + 2.0 ** -8 * 0.5 * 1e-3)
