"""What this library is timed on: training steps and forward passes of LIF-SNNs through its public entry points.

A case is one network with one batch of spike trains and one way of calling the library:

  call      "train": bind the batch, one snn_bptt step, logits, loss and every gradient out; "infer": snn_forward and the
            logits.
  strategy  state storage of the training step (with its coarse and fine interval; 0 = the library's default) under
            `budget` bytes of HBM for activations (0 = no limit).
  push      the step begins by handing over every weight matrix, as a training loop does after each optimiser step; without
            it the weights stay as they are (several batches per optimiser step, evaluation).
  host      the spike trains come from a data loader in host memory; without it they are on the GPU.
  window, tier   compact support of the surrogate derivative (0 = none); 1 = spike bitmasks of finished segments on the host.

The spike trains are Bernoulli bytes [T][B][n_in] at rate p_in, the labels uniform; weights are normal with the standard
deviation gain * 2 / sqrt(fan_in * rate), as this repository's synthetic workloads draw them (rate: p_in for the first
matrix, 0.05 behind a hidden layer).  gain 1 makes the hidden layers fire at 40-50 %, gains near 0.2 at about 5 %.  `rate` is
what the hidden layers are expected to fire at; only the count of operations in work() uses it.

Everything is made on the GPU from the seed.  Gradients are copied into tensors on the GPU that the state holds, where an
optimiser would read them.
"""
import math

import torch

import paper_2412_11810_amd as snn

STRATEGIES = {"standard": snn.SNN_STANDARD, "chunk": snn.SNN_CHUNK, "remote": snn.SNN_REMOTE, "double": snn.SNN_DOUBLE,
              "hier": snn.SNN_HIER}
P_HIDDEN = 0.05  # rate that the weight scale assumes behind a hidden layer


def _case(name, n_in, hidden, n_out, T, B, p_in, gain, rate, call="train", strategy="standard", coarse=0, fine=0, budget=0,
          density=1.0, push=False, host=False, window=0.0, tier=0):
    c = dict(n_in=n_in, hidden="-".join(str(n) for n in hidden), n_out=n_out, T=T, B=B, p_in=p_in, gain=gain, rate=rate,
             call=call, strategy=strategy, coarse=coarse, fine=fine, budget=budget, density=density, push=push, host=host,
             window=window, tier=tier)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one training step of a 64-neuron network over 50 steps; launches and host work count
        _case("tiny_chunk", 32, [64], 10, 50, 2, 0.05, 1.0, 0.5, strategy="chunk", fine=10),
        # evaluation of a two-layer classifier on a batch that a data loader has put into host memory
        _case("classifier_infer_host", 700, [256, 256], 20, 1000, 32, 0.02, 1.0, 0.45, call="infer", host=True),
        # a step of that classifier's training loop, all states stored: new weights, batch, gradients
        _case("classifier_standard_loop", 700, [256, 256], 20, 1000, 32, 0.02, 1.0, 0.45, push=True),
        # the same network with its checkpoints in host memory
        _case("classifier_remote", 700, [256, 256], 20, 1000, 32, 0.02, 1.0, 0.45, strategy="remote", coarse=32),
        # a small network whose sizes fit no tile: odd widths, batch, sequence length; batched transfers to the host
        _case("ragged_hier_loop", 90, [200, 75], 11, 333, 13, 0.04, 1.0, 0.45, strategy="hier", coarse=4, fine=17, push=True,
              host=True),
        # evaluation of a wide three-layer network at low activity
        _case("wide_infer", 700, [1024, 1024, 1024], 20, 500, 64, 0.01, 0.156, 0.05, call="infer"),
        # training of that network under a budget, coarse checkpoints on the host and fine ones in HBM
        _case("wide_double", 700, [1024, 1024, 1024], 20, 1000, 64, 0.01, 0.156, 0.05, strategy="double", coarse=100, fine=10,
              budget=8_000_000_000),
        # wide layers at widths that fit no tile, every synapse present, a training loop
        _case("ragged_wide_chunk_loop", 300, [1500, 1100], 20, 150, 24, 0.02, 0.18, 0.05, strategy="chunk", push=True),
        # a long sequence at high activity
        _case("long_double", 128, [512, 512], 10, 4000, 16, 0.01, 1.0, 0.45, strategy="double", coarse=316, fine=18,
              budget=4_000_000_000),
        # a masked network with a windowed surrogate and its spike trains on the host tier, a training loop
        _case("masked_window_loop", 512, [2048, 2048], 20, 2000, 16, 0.02, 0.21, 0.05, strategy="remote", coarse=50, density=0.1,
              push=True, window=0.5, tier=1),
        # the largest network: 33 thousand neurons, recurrent matrices 90 % zero, at 5 % activity ...
        _case("large_double", 1024, [8192] * 4, 100, 512, 32, 0.02, 0.2175, 0.05, strategy="double", coarse=512, fine=64,
              budget=32_000_000_000, density=0.1),
        # ... and at about 20 %, over a shorter sequence
        _case("large_active", 1024, [8192] * 4, 100, 200, 32, 0.02, 0.316, 0.2, strategy="double", coarse=50, fine=10,
              budget=32_000_000_000, density=0.1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A layer width: half of them multiples of 64, the others as they come."""
    n = _log_int(rng, lo, hi)
    return max(lo, n // 64 * 64) if rng.random() < 0.5 else n


def _draw(rng):
    size = rng.choice(["narrow", "middle", "wide"])
    n_in, n_out = _log_int(rng, 32, 1024), _log_int(rng, 2, 100)
    p_in = rng.choice([0.01, 0.02, 0.05])
    gain, rate = rng.choice([(1.0, 0.45), (0.2, 0.05), (0.17, 0.03)])
    density, window, tier = 1.0, 0.0, 0
    if size == "narrow":
        hidden = [_width(rng, 32, 256) for _ in range(rng.randint(1, 3))]
        T, B = _log_int(rng, 40, 2000), _log_int(rng, 1, 64)
    elif size == "middle":
        hidden = [_width(rng, 257, 1024) for _ in range(rng.randint(1, 3))]
        T, B = _log_int(rng, 40, 1500), _log_int(rng, 4, 64)
    else:
        hidden = [_width(rng, 1025, 8192)] * rng.randint(1, 4) if rng.random() < 0.5 else \
            [_width(rng, 1025, 4096) for _ in range(rng.randint(1, 3))]
        T, B = _log_int(rng, 20, 160), _log_int(rng, 8, 32)
        if max(hidden) > 2048 or rng.random() < 0.5:
            density = rng.choice([0.05, 0.1, 0.2])
        gain, rate = rng.choice([(0.2175, 0.05), (0.17, 0.02), (0.3, 0.15)])
        window = rng.choice([0.0, 0.0, 0.0, 0.5])
    call = rng.choice(["infer", "train", "train", "train"])
    if call == "infer":
        return _case(None, n_in, hidden, n_out, T, B, p_in, gain, rate, call="infer", density=density, host=rng.random() < 0.5)
    strategy = rng.choice(list(STRATEGIES))
    coarse = fine = 0
    if strategy == "chunk":
        fine = rng.choice([0, _log_int(rng, 8, 64)])
    elif strategy == "remote":
        coarse = rng.choice([0, _log_int(rng, 8, 64)])
        tier = rng.choice([0, 0, 1])
    elif strategy == "double" and rng.random() < 0.7:
        coarse = min(T, _log_int(rng, 20, 400))
        fine = rng.randint(1, max(1, coarse // 2))
        fine = max(fine, min(8, coarse))
    elif strategy == "hier" and rng.random() < 0.7:
        coarse, fine = rng.randint(2, 6), min(T, _log_int(rng, 8, 64))
    return _case(None, n_in, hidden, n_out, T, B, p_in, gain, rate, strategy=strategy, coarse=coarse, fine=fine,
                 budget=rng.choice([0, 0, 32_000_000_000]), density=density, push=rng.random() < 0.5, host=rng.random() < 0.25,
                 window=window, tier=tier)


def draw(rng):
    most = [work(c) for c in listed()]
    top_b, top_f = max(w["bytes"] for w in most), max(w["flops"] for w in most)
    while True:
        c = _draw(rng)
        w = work(c)
        if w["bytes"] <= top_b and w["flops"] <= top_f:
            return c


def _hidden(case):
    return [int(n) for n in case["hidden"].split("-")]


class _Net(snn.Snn):
    """The library's context with gradients copied to the GPU (the C entry point takes host or device memory)."""

    def grads_to(self, kind, layer, dst):
        self._check(snn.lib().snn_grads(self._h, kind, layer, dst.data_ptr(), dst.numel()))


def prepare(case, seed):
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed) * 7919 + 11)
    hidden, T, B = _hidden(case), case["T"], case["B"]
    pre = [case["n_in"]] + hidden[:-1]

    def normal(rows, cols, p):
        w = torch.randn((rows, cols), generator=g, device=dev, dtype=torch.float32)
        return w.mul_(case["gain"] * 2.0 / math.sqrt(rows * p))

    W = []  # (kind, layer, weights, mask)
    for l, n in enumerate(hidden):
        W.append((snn.SNN_W_IN, l, normal(pre[l], n, case["p_in"] if l == 0 else P_HIDDEN), None))
        w, mask = normal(n, n, P_HIDDEN), None
        if case["density"] < 1.0:
            mask = (torch.rand((n, n), generator=g, device=dev) < case["density"]).to(torch.uint8)
            w.mul_(mask)
        W.append((snn.SNN_W_REC, l, w, mask))
    W.append((snn.SNN_W_OUT, 0, normal(hidden[-1], case["n_out"], P_HIDDEN), None))
    x = torch.empty((T, B, case["n_in"]), dtype=torch.uint8, device=dev)
    x.copy_(torch.rand(x.shape, generator=g, device=dev) < case["p_in"])
    y = torch.randint(0, case["n_out"], (B,), generator=g, device=dev, dtype=torch.int32)
    if case["host"]:
        x, y = x.cpu().numpy(), y.cpu().numpy()
    net = _Net(snn.make_config(case["n_in"], hidden, case["n_out"], T, B, surr_window=case["window"], spike_tier=case["tier"]))
    torch.cuda.synchronize()
    for kind, layer, w, mask in W:
        net.snn_set_weights(kind, layer, w, mask)
    grads = [torch.empty_like(w) for _, _, w, _ in W] if case["call"] == "train" else []
    return dict(case=case, net=net, W=W, x=x, y=y, grads=grads)


def run(state):
    case, net = state["case"], state["net"]
    if case["call"] == "infer":
        loss = net.snn_forward(state["x"], state["y"], case["T"])
        ubar, _ = net.snn_get_readout()
        return dict(loss=loss, ubar=ubar)
    if case["push"]:
        for kind, layer, w, mask in state["W"]:
            net.snn_set_weights(kind, layer, w, mask)
    net.snn_bind_inputs(state["x"], state["y"], case["T"])
    net.snn_bptt(STRATEGIES[case["strategy"]], case["coarse"], case["fine"], case["budget"], want_stats=False)
    ubar, loss = net.snn_get_readout()
    for (kind, layer, _, _), dst in zip(state["W"], state["grads"]):
        net.grads_to(kind, layer, dst)
    return dict(loss=loss, ubar=ubar, grads=state["grads"])


def work(case):
    """Each input read once (spike bytes, weights, masks), each output written once; operations of the event-driven method:
    one add per spike and existing synapse in the forward pass and again in the weight gradients, two operations per existing
    synapse, step and batch element for every product with a transposed matrix (the surrogate has no compact support), ten per
    neuron, step and batch element and pass for the neuron itself."""
    hidden, B, T = _hidden(case), case["B"], case["T"]
    pre = [case["n_in"]] + hidden[:-1]
    weights = masks = events = products = 0.0
    for l, n in enumerate(hidden):
        rate_in = case["p_in"] if l == 0 else case["rate"]
        syn_in, syn_rec = pre[l] * n, n * n * case["density"]
        weights += syn_in + n * n
        masks += n * n if case["density"] < 1.0 else 0
        events += rate_in * syn_in + case["rate"] * syn_rec
        products += 2.0 * (syn_rec + (syn_in if l > 0 else 0))
    out = hidden[-1] * case["n_out"]
    weights += out
    events += case["rate"] * out
    products += 2.0 * out
    steps, neuron = float(B) * T, 10.0 * sum(hidden)
    read = float(T) * B * case["n_in"] + 4 * B + 4 * weights + (masks if case["push"] else 0)
    if case["call"] == "infer":
        return {"bytes": read + 4 * B * case["n_out"] + 4, "flops": steps * (events + neuron)}
    return {"bytes": read + 4 * weights + 4 * B * case["n_out"] + 4, "flops": steps * (2 * events + products + 2 * neuron)}


def tolerance(case):
    # Spike trains are exact, so logits and loss only differ by sums of the readout (kept in 64 bits) rounded to 32.  Gradients
    # are 32-bit products and sums of one step, added over the steps in 64 bits: with the sums over the postsynaptic neurons
    # taken in two other orders they differ by 1e-7 (512 and 1024 neurons wide) to 5.3e-7 (four layers of 8192), single values
    # by up to 1.4e-5.  Four times that.
    return {"rel": 2e-6, "max": 6e-5}
