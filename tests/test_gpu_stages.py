"""Per-stage GPU parity of the backbone kernels against the oracle's stage
outputs: patch embedding, attention + projection residual, MLP residual
(fusion_debug_state stops the pipeline after a stage of block 1)."""
import numpy as np
import pytest

from oracle import fusion_oracle as fo
import parity_utils as pu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _oracle_stage(cfg, Wp, img, stage, mode):
    x = fo.patch_embed(img, Wp, cfg, mode)
    if stage == 0:
        return x
    Wb = fo._b_weights(Wp, 1)
    s = np.ones(x.shape[0], np.float32)
    if stage == 1:
        O, _ = fo.attention(x, s, Wb, cfg, mode, False)
        return x + (O @ Wb["proj_w"].T + Wb["proj_b"])
    return fo.block(x, s, Wb, cfg, mode)[0]


@pytest.mark.parametrize("name,batch,tol", [("tiny", 8, 1e-4), ("deit_ti", 6, 2e-2),
                                            ("deit_s", 4, 2e-2), ("deit_b", 2, 2e-2),
                                            ("deit_s_384", 2, 2e-2)])
@pytest.mark.parametrize("stage", [0, 1, 2])
def test_block1_stage_parity(torch_cuda, name, batch, tol, stage):
    torch = torch_cuda
    cfg, W, imgs = pu.make(name, batch=batch, affine="random")
    print(f"[stage parity] {name} B={batch} stage={stage}", flush=True)
    model = pu.gpu_model(cfg, W, batch)
    xs, live = model.debug_state(torch.from_numpy(imgs).cuda(), 1, stage)
    assert list(live) == list(range(batch))
    mode = pu.mode_of(cfg)
    Wp = fo.prepare_weights(W, mode)
    worst = 0.0
    for i in range(batch):
        ref = _oracle_stage(cfg, Wp, imgs[i], stage, mode)
        assert xs[i].shape == ref.shape
        err = float(np.abs(xs[i] - ref).max())
        worst = max(worst, err)
        assert err <= tol, (i, err)
    print(f"  max |dx| = {worst:.3e}")


@pytest.mark.parametrize("routers,rho,delta", [("closed", 1.5, 1.0), ("open", 1.0, 1.0),
                                               ("bias", 0.5, 0.1)])
def test_rows_far_from_those_expected(routers, rho, delta):
    """The GEMM kernels are chosen for the rows that the routers give at their
    bias and for all samples live.  Routers that merge nothing or all they may,
    and samples that leave early, give each image the bits of a run of its own."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg, W, imgs = pu.make("deit_ti", affine="random")
    B = 40
    x = torch.from_numpy(imgs[:B]).cuda()
    B = x.shape[0]
    if routers != "bias":
        for b in cfg["merges"]:  # each block's CLS rows point along their mean
            m = pu.gpu_model(cfg, W, 4)
            m.set_exit_thresholds([1.0] * len(cfg["exits"]))
            mu = np.stack([s[0] for s in m.debug_state(x[:4].contiguous(), b, 2)[0]]).mean(0)
            m.close()
            W[f"blk{b}.router_w"] = ((-40 if routers == "closed" else 40) * mu
                                     / np.dot(mu, mu)).astype(np.float32)
    out = []
    for n in (B, 1):
        m = pu.gpu_model(cfg, W, n)
        m.set_exit_thresholds([delta] * len(cfg["exits"]))
        m.set_router_strength(rho)
        runs = [[t.clone() for t in m.run(x[i:i + n].contiguous())] for i in range(0, B, n)]
        out.append([torch.cat(t) for t in zip(*runs)])
        torch.cuda.synchronize()
        m.close()
    print(f"[rows] routers {routers} rho {rho}: tokens {out[0][2][0].tolist()}, "
          f"{int((out[0][1] < cfg['L']).sum())} of {B} leave early", flush=True)
    for a, b in zip(*out):
        assert torch.equal(a, b)
