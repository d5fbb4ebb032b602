"""A U-Net training step recorded into a HIP graph on a stream of its own and replayed on the default stream: reading the weights and a
gradient right behind the replay, with no wait between, gives those of the replayed steps, bit for bit those of the same steps run eagerly."""
import numpy as np
import pytest
import torch

import sk_synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_reads_wait_for_replays_on_the_default_stream(dtype):
    from paper_1509_03371_amd import binding as B
    h = w = 188
    img = torch.from_numpy(S.uniform_image(1, 1, h, w, 3)).cuda()
    nets = []
    for _ in range(2):
        net = B.UNet(1, 2, dtype=dtype)                # its largest tensors are 37.7 MB: many pieces of the reader's
        rng = np.random.default_rng(5)
        for i in range(net.num_params()):
            s = net.param_shape(i)
            net.set_weights(i, (rng.standard_normal(s, dtype=np.float32) * np.sqrt(2.0 / (s[1] * s[2] * s[3]))).astype(np.float32))
        net.plan(1, h, w, training=True)
        nets.append(net)
    eager, replayed = nets
    ho, wo = eager.output_size(h, w)
    labels = torch.from_numpy(S.binary_labels(1, ho, wo, 4)).cuda()
    prob, loss = torch.empty((1, 2, ho, wo), device="cuda"), torch.empty(1, device="cuda")

    def step(net, stream):
        net.forward(img, prob, stream)
        net.backward(labels, loss, stream)
        net.sgd_step(1e-2, 0.9, stream=stream)

    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            step(replayed, torch.cuda.current_stream())
    torch.cuda.synchronize()
    read = [i for i in range(eager.num_params()) if np.prod(eager.param_shape(i)) >= 1 << 21]
    assert len(read) >= 4 and any(eager.param_shape(i)[2] == 2 for i in read)      # an up-convolution, which is turned on the device, among them
    for rep in range(3):
        for _ in range(2):
            step(eager, torch.cuda.current_stream())
        want = [eager.get_weights(i) for i in read], eager.get_grad(read[-1])
        for _ in range(2):
            graph.replay()
        got = [replayed.get_weights(i) for i in read], replayed.get_grad(read[-1])
        for a, b in zip(want[0] + [want[1]], got[0] + [got[1]]):
            assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), rep
    for net in nets:
        net.close()
