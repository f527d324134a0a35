"""The network's convolution, data-gradient and weight-gradient kernels at the edges of their
tiles and dispatch rules, against the same network composed of torch operations on the GPU in
FP32, rounded to BF16 where the library rounds (activations, weights, gradients entering a
layer)."""
import numpy as np
import pytest

from paper_1901_08269_amd import learned

pytestmark = pytest.mark.gpu

# Both sides round to BF16 at the same places and sum in FP32 in different orders, so a stored
# value can differ by one unit in the last place (2^-8 relative): 1e-2 of a tensor's maximum for
# the prediction, twice that for gradients, which pass through the network twice.
PRED_BAR, GRAD_BAR, LOSS_BAR = 1e-2, 2e-2, 2e-3


def _bf(t):
    import torch
    return t.to(torch.bfloat16).float()


def _shapes(ch):
    ci = [3, ch[0], ch[0], ch[1], ch[1], ch[2], ch[2], ch[3], ch[3] + ch[2], ch[2], ch[2] + ch[1], ch[1],
          ch[1] + ch[0], ch[0]]
    co = [ch[0], ch[0], ch[1], ch[1], ch[2], ch[2], ch[3], ch[3], ch[2], ch[2], ch[1], ch[1], ch[0], ch[0]]
    return list(zip(co, ci))


def _taps(x):
    """The 27 shifted copies of x (ci, n, n, n) with zero padding, as (tap, (ci, n, n * n))."""
    import torch
    n = x.shape[-1]
    p = torch.nn.functional.pad(x, (1, 1, 1, 1, 1, 1))
    for t in range(27):
        a, b, c = t // 9, (t // 3) % 3, t % 3
        yield t, p[:, a:a + n, b:b + n, c:c + n].reshape(x.shape[0], n, n * n)


def _conv(x, w):
    n = x.shape[-1]
    y = 0
    for t, s in _taps(x):
        y = y + w[:, :, t].contiguous() @ s.reshape(s.shape[0], -1)
    return y.view(-1, n, n, n)


def _wgrad(x, g):
    """sum_v g[co] x[v + tap][ci], one plane after another"""
    import torch
    gz = g.view(g.shape[0], g.shape[1], -1).permute(1, 0, 2).contiguous()             # (z, co, n^2)
    out = []
    for _, s in _taps(x):
        out.append(torch.bmm(gz, s.permute(1, 2, 0).contiguous()).sum(0))
    return torch.stack(out, dim=2)


def _network(w, ch, inp, tgt):
    """(prediction, loss, gradient) with the library's roundings."""
    import torch
    par, off, sl = [], 0, []
    flat = torch.as_tensor(w, device="cuda")
    for co, ci in _shapes(ch):
        n = 27 * co * ci
        par.append((_bf(flat[off:off + n]).view(co, ci, 27), flat[off + n:off + n + co]))
        sl.append((slice(off, off + n), slice(off + n, off + n + co)))
        off += n + co
    hw = flat[off:]
    grad = torch.zeros_like(flat)
    preds, loss = [], 0.0
    for b in range(inp.shape[0]):
        ins, outs = [None] * 14, [None] * 14

        def layer(q, x):
            ins[q] = x
            wq, bq = par[q]
            outs[q] = _bf(torch.relu(_conv(x, wq) + bq.view(-1, 1, 1, 1)))
            return outs[q]

        def pool(x):
            c, n = x.shape[0], x.shape[-1] // 2
            return _bf(x.view(c, n, 2, n, 2, n, 2).sum(dim=(2, 4, 6)) * 0.125)

        def up(x):
            return x.repeat_interleave(2, 1).repeat_interleave(2, 2).repeat_interleave(2, 3)

        x = _bf(inp[b])
        for q in range(8):
            x = layer(q, pool(x) if q in (2, 4, 6) else x)
        for q, sk in ((8, 5), (10, 3), (12, 1)):
            x = layer(q + 1, layer(q, torch.cat([up(x), outs[sk]])))
        p = (x * hw[:-1].view(-1, 1, 1, 1)).sum(0) + hw[-1]
        preds.append(p)
        d = p.double() - tgt[b].double()
        loss += float((d * d).sum() / tgt.numel())
        dp = (2.0 * d / tgt.numel()).float()
        grad[off:-1] += (outs[13] * dp).sum(dim=(1, 2, 3))
        grad[-1] += dp.sum()
        gout = [None] * 14
        gout[13] = dp * hw[:-1].view(-1, 1, 1, 1)
        for q in range(13, -1, -1):
            gb = _bf(torch.where(outs[q] > 0, gout[q], torch.zeros_like(gout[q])))
            grad[sl[q][0]] += _wgrad(ins[q], gb).reshape(-1)
            grad[sl[q][1]] += gb.sum(dim=(1, 2, 3))
            if q == 0:
                break
            gi = _conv(gb, par[q][0].permute(1, 0, 2).flip(2).contiguous())
            if q in (2, 4, 6):
                gout[q - 1] = gout[q - 1] + up(gi) * 0.125
            elif q in (8, 10, 12):
                c0, m = outs[q - 1].shape[0], gi.shape[-1] // 2
                gout[q - 1] = gi[:c0].reshape(c0, m, 2, m, 2, m, 2).sum(dim=(2, 4, 6))
                gout[{8: 5, 10: 3, 12: 1}[q]] = gi[c0:]
            else:
                gout[q - 1] = gi
    return torch.stack(preds), loss, grad.cpu().numpy(), sl, off


# 8: the coarsest level has one cell; 24: levels of 24, 12, 6 and 3 cells, 16 channels
# everywhere (every weight gradient split over the waves' steps); 40: four output groups, and
# five input groups on one output group; 264: rows too long for one range of staged voxels
@pytest.mark.parametrize("nc,B,ch", [(8, 3, (16, 32, 48, 64)), (24, 1, (16, 16, 16, 16)), (40, 2, (16, 64, 64, 64)),
                                     (264, 1, (16, 32, 48, 64))])
def test_network_kernels_match_torch(nc, B, ch):
    import torch
    print(f"[case] network kernels nc={nc} B={B} channels={ch}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(nc)
    inp = torch.randn((B, 3, nc, nc, nc), generator=gen, device="cuda")
    tgt = torch.randn((B, nc, nc, nc), generator=gen, device="cuda")
    m = learned.Model(nc, batch=B, channels=ch, seed=4)
    pred = m.forward(inp)
    loss = m.train_step(inp, tgt, update=False)
    w, g = m.params(grads=True)
    m.close()
    p_ref, l_ref, g_ref, sl, off = _network(w, ch, inp, tgt)
    dp = float((pred - p_ref).abs().max() / p_ref.abs().max())
    print(f"prediction {dp:.2e}, loss {loss:.6e} / {l_ref:.6e}", flush=True)
    assert dp <= PRED_BAR
    assert abs(loss - l_ref) <= LOSS_BAR * abs(l_ref)
    for q, parts in enumerate(sl + [(slice(off, None),)]):
        for part in parts:
            err = float(np.max(np.abs(g[part] - g_ref[part])) / np.max(np.abs(g_ref[part])))
            assert err <= GRAD_BAR, (q, err)
