"""Host-side checks of the screen's training (torch tensors on the CPU, so not
among the files that run under the sanitizers)."""
import numpy as np

import paper_2502_08673_amd as tt


def test_training_step_uses_the_buffers_that_the_net_holds(monkeypatch):
    """A buffer that a program puts in another's place (a loss kept per step,
    a tensor's new storage) is the one that the step in one call gets: the
    replaced one may be freed."""
    import torch

    sc = tt.screen
    monkeypatch.setattr(sc, "cast_bf16", lambda x, y: None)
    seen = []

    def step(state, *rest):
        seen.append({k: (list(v) if hasattr(v := getattr(state, k), "__len__") else v) for k, _ in state._fields_})

    monkeypatch.setattr(sc, "mlp_train_step", step)
    params = [(np.zeros((sc.DIMS[i + 1], sc.DIMS[i]), np.float32), np.zeros(sc.DIMS[i + 1], np.float32))
              for i in range(4)]
    net = sc.ScreenNet(params, max_batch=64, device="cpu")
    args = [torch.zeros((64, 32), dtype=torch.int16)] + [torch.zeros((64, k)) for k in (8, 8, 4)]
    assert net.train_step(*args, 64, 1e-3) is net.loss
    old = (net.loss, net.z, net.scratch, net.dh[1])  # kept, so that the new ones lie elsewhere
    net.loss, net.z, net.scratch, net.dh[1] = (t.clone() for t in old)
    w0 = net.W32[0].data_ptr()
    net.W32[0].data = net.W32[0].data.clone()
    assert net.train_step(*args, 64, 1e-3) is net.loss
    assert seen[0]["loss"] == old[0].data_ptr() and seen[0]["pw"][0] == w0
    assert seen[1]["loss"] == net.loss.data_ptr() != old[0].data_ptr()
    assert seen[1]["z"] == net.z.data_ptr() and seen[1]["scratch"] == net.scratch.data_ptr()
    assert seen[1]["dh"][1] == net.dh[1].data_ptr() and seen[1]["pw"][0] == net.W32[0].data_ptr() != w0
    assert seen[1]["act"] == seen[0]["act"] and seen[1]["scratch_floats"] == net.scratch.numel()
