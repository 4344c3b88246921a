"""The work that users of the library have it do, as cases that can be timed: each case is built by `prepare`, run once by
`run` through the public binding, and priced by `work`.

The configurations are the named ones of synth/inputs.py (BERT-base and decoder shaped layers, 64 to 10 000 tenants, up to
512 requests of up to 512 tokens in a batch) and their small ends: a handful of requests, a few hundred rows.  Inputs are
drawn here, from the seed alone: hidden states N(0, 1), weights and biases N(0, 0.02), LayerNorm gains 1 + N(0, 0.02),
tenant ids uniform or Zipf over the id space.  Sequence lengths are spread evenly over [len_min, len_max] in random order,
so that the number of rows belongs to the case and not to the seed.

Fields of a case
  use       "forward"   one call over a batch (every request's own tenant's layers)
            "serve"     aggregate of looked-up representations, the shared layers with the tenants' adapters, output heads
            "generate"  prompts into the key/value cache, then `steps` decode steps of one token per request
            "queue"     requests pushed one by one into the request queue, `batches` full batches run, every result fetched
  block     the layer kind; dtype, d, ff, layers, rank: its sizes
  tenants   id space; slots: tenants resident in HBM (0 = all of them; otherwise a host tier holds them all)
  requests  per batch; zipf: exponent of the tenants' popularity (0 = uniform)
"""
import math

import numpy as np
import torch

import paper_2504_17449_amd as hmi

BLOCKS = {"ffn": hmi.HMI_BLOCK_FFN, "encoder": hmi.HMI_BLOCK_ENC_POSTLN, "decoder": hmi.HMI_BLOCK_DEC_PRELN,
          "adapter": hmi.HMI_BLOCK_ADAPTER, "shared_encoder": hmi.HMI_BLOCK_ENC_ADAPTER,
          "shared_decoder": hmi.HMI_BLOCK_DEC_ADAPTER}
RANK = 64            # bottleneck width of an adapter
CLASSES = 32         # widest output head
TABLE = 5000         # entries of the table of precomputed representations
MASTER = 1 << 23     # normal draws that all weights of a state are windows of
IMAGES = 256         # distinct weight sets behind a host tier; the other ids share them


def _case(name, use, block, dtype, d, ff, layers, tenants, requests, len_min, len_max, zipf=0.0, steps=0, batches=1, slots=0):
    case = {"use": use, "block": block, "dtype": dtype, "d": d, "ff": ff, "layers": layers, "tenants": tenants,
            "slots": slots, "requests": requests, "len_min": len_min, "len_max": len_max, "zipf": zipf, "steps": steps,
            "batches": batches}
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest call: four tenants' 64-wide FFN blocks over 128 rows, fp32 (latency, launches)
        _case("ffn_f32_tiny", "forward", "ffn", "f32", 64, 256, 1, 4, 8, 16, 16),
        # fp32 storage at BERT-base width: a batch of 24 ragged requests through eight tenants' encoder layers
        _case("encoder_f32", "forward", "encoder", "f32", 768, 3072, 2, 8, 24, 16, 128),
        # every tenant owns an FFN block: the default benchmark batch
        _case("ffn_tenants", "forward", "ffn", "bf16", 768, 3072, 1, 64, 256, 128, 128),
        # every tenant owns two encoder layers, popularity heavily skewed
        _case("encoder_tenants", "forward", "encoder", "bf16", 768, 3072, 2, 1000, 512, 128, 128, zipf=1.1),
        # every tenant owns a decoder layer: ragged prompts, then a few tokens each
        _case("decoder_generate", "generate", "decoder", "bf16", 1024, 4096, 1, 2000, 256, 32, 512, zipf=1.0, steps=8),
        # the bottleneck adapter alone
        _case("adapter", "forward", "adapter", "bf16", 768, RANK, 1, 1000, 512, 128, 128, zipf=1.1),
        # the whole request path of the serving layer (six shared layers, tenant adapters, heads): a full batch,
        _case("serve_full", "serve", "shared_encoder", "bf16", 768, 3072, 6, 1000, 512, 128, 128, zipf=1.1),
        # an ordinary batch as it comes in, ragged,
        _case("serve_ordinary", "serve", "shared_encoder", "bf16", 768, 3072, 6, 1000, 37, 16, 128, zipf=1.1),
        # and two requests on an idle server
        _case("serve_two", "serve", "shared_encoder", "bf16", 768, 3072, 6, 1000, 2, 40, 101, zipf=1.1),
        # generation through six shared decoder layers with tenant adapters: a full batch of ragged prompts,
        _case("generate_full", "generate", "shared_decoder", "bf16", 768, 3072, 6, 1000, 256, 32, 512, zipf=1.0, steps=16),
        # and a few conversations
        _case("generate_few", "generate", "shared_decoder", "bf16", 768, 3072, 6, 1000, 7, 16, 200, zipf=1.0, steps=16),
        # 10 000 tenants' adapters in host memory behind an HBM cache: requests through the queue, each batch new
        _case("queue_10k", "queue", "shared_encoder", "bf16", 768, 3072, 6, 10000, 512, 16, 256, zipf=0.8, batches=4, slots=1024),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: sizes spread over their logarithm, odd ones among them."""
    kind = rng.choice(["f32", "own", "own", "adapter", "serve", "serve", "generate", "generate", "queue"])
    lo = rng.randint(1, 64)
    hi = max(lo, _log_int(rng, 16, 512))
    zipf = rng.choice([0.0, 0.8, 1.0, 1.1])
    if kind == "f32":
        d = rng.choice([64, 128, 192, 256, 512, 768])
        layers = rng.randint(1, 2)
        return _case("", "forward", rng.choice(["ffn", "encoder", "decoder"]), "f32", d, 4 * d, layers,
                     _log_int(rng, 1, 16), _log_int(rng, 1, 32), min(lo, 16), min(hi, 128), zipf)
    if kind == "own":
        d = rng.choice([320, 512, 768, 768, 1024])
        requests = _log_int(rng, 1, 256)
        return _case("", "forward", rng.choice(["ffn", "encoder", "decoder"]), "bf16", d, 4 * d, rng.randint(1, 2),
                     _log_int(rng, 1, 256), requests, lo, min(hi, max(lo, 40000 // requests)), zipf)
    if kind == "adapter":
        return _case("", "forward", "adapter", "bf16", rng.choice([256, 512, 768]), RANK, 1, _log_int(rng, 1, 1000),
                     _log_int(rng, 1, 512), min(lo, 128), min(hi, 128) if hi > lo else lo, zipf)
    if kind == "serve":
        d = rng.choice([512, 768, 768])
        requests = _log_int(rng, 1, 400)
        lo = max(lo, -(-100 // requests))      # a hundred rows at least: one label in the balance is one in a hundred
        return _case("", "serve", "shared_encoder", "bf16", d, 4 * d, rng.randint(2, 6), _log_int(rng, 1, 1000), requests, lo,
                     max(lo, min(hi, 128)), zipf)
    if kind == "generate":
        block = rng.choice(["decoder", "shared_decoder", "shared_decoder"])
        d = 1024 if block == "decoder" else 768
        return _case("", "generate", block, "bf16", d, 4 * d, 1 if block == "decoder" else rng.randint(2, 6),
                     _log_int(rng, 1, 1000), _log_int(rng, 1, 200), lo, hi, zipf, steps=rng.randint(4, 16))
    requests = _log_int(rng, 24, 400)
    return _case("", "queue", "shared_encoder", "bf16", 768, 3072, rng.randint(2, 6), 10000, requests, lo, min(hi, 200) if hi > lo else lo,
                 0.8, batches=rng.randint(2, 4), slots=2 * requests)


# ---------------------------------------------------------------- sizes

def _lens(case):
    """The case's sequence lengths in ascending order."""
    r, lo, hi = case["requests"], case["len_min"], max(case["len_min"], case["len_max"])
    return [lo + int(round((hi - lo) * i / max(1, r - 1))) for i in range(r)]


def _popularity(case):
    k = np.arange(1, case["tenants"] + 1, dtype=np.float64)
    p = k ** -case["zipf"] if case["zipf"] else np.ones_like(k)
    return p / p.sum()


def _own_shapes(case):
    """Tensors of one (tenant, layer) in canonical order: (shape, kind)."""
    d, f = case["d"], case["ff"]
    if case["block"] == "adapter":
        return [((f, d), "w"), ((f,), "b"), ((d, f), "w"), ((d,), "b")]
    if case["block"] in ("shared_encoder", "shared_decoder"):
        return [((RANK, d), "w"), ((RANK,), "b"), ((d, RANK), "w"), ((d,), "b")]
    ffn = [((f, d), "w"), ((f,), "b"), ((d, f), "w"), ((d,), "b"), ((d,), "g"), ((d,), "b")]
    if case["block"] == "ffn":
        return ffn
    return [((3 * d, d), "w"), ((3 * d,), "b"), ((d, d), "w"), ((d,), "b"), ((d,), "g"), ((d,), "b")] + ffn


def _shared_shapes(case):
    return _own_shapes(dict(case, block="encoder")) if case["block"].startswith("shared") else []


def _elements(shapes):
    return sum(int(np.prod(s)) for s, _ in shapes)


def work(case):
    e = 4 if case["dtype"] == "f32" else 2
    d, f, layers, steps, batches = case["d"], case["ff"], case["layers"], case["steps"], case["batches"]
    lens = _lens(case)
    r, n = len(lens), sum(lens)
    distinct = float(np.sum(1.0 - (1.0 - _popularity(case)) ** r))
    weights = e * layers * (distinct * _elements(_own_shapes(case)) + _elements(_shared_shapes(case)))
    if case["block"] in ("ffn", "adapter"):
        linear = 4 * d * f
    else:
        linear = 8 * d * d + 4 * d * f + (4 * d * RANK if case["block"].startswith("shared") else 0)
    flops, moved = n * linear * layers, weights + 2 * n * d * e
    causal = case["block"] in ("decoder", "shared_decoder")
    if case["block"] not in ("ffn", "adapter"):
        flops += layers * sum(4 * s * d * ((s + 1) / 2 if causal else s) for s in lens)
    if case["use"] == "serve":
        moved += min(3 * n * d, 3 * TABLE * d) * e - n * d * e + n * 4          # table rows and ids instead of x
        moved += n * (CLASSES * 4 + 4) + distinct * CLASSES * d * e
        flops += n * 5 * d + r * 2 * d * CLASSES
    if case["use"] == "generate":
        moved += layers * n * 2 * d * e                                          # keys and values written
        for i in range(steps):
            moved += weights + 2 * r * d * e + layers * 2 * d * e * (n + r * (i + 1))
            flops += layers * (r * linear + 4 * d * (n + r * (i + 1)))
    return {"bytes": float(moved * batches), "flops": float(flops * batches)}


# ---------------------------------------------------------------- inputs

class _Draws:
    """Weights of one state: windows of one seeded sequence of normal draws, as the host arrays a pool is loaded from."""

    def __init__(self, case, seed):
        self.f32 = case["dtype"] == "f32"
        g = torch.Generator(device="cuda").manual_seed(seed)
        z = torch.randn(MASTER, generator=g, device="cuda") * 0.02
        self.small = self._host(z)
        self.gains = self._host(1.0 + z[: 1 << 16])
        self.rng = np.random.default_rng(seed)

    def _host(self, z):
        return z.cpu().numpy() if self.f32 else z.to(torch.bfloat16).view(torch.int16).cpu().numpy().view(np.uint16)

    def tensor(self, shape, kind):
        src = self.gains if kind == "g" else self.small
        n = int(np.prod(shape))
        off = int(self.rng.integers(0, src.shape[0] - n))
        return src[off:off + n].reshape(shape)

    def tensors(self, shapes):
        return [self.tensor(s, k) for s, k in shapes]


def _normal(shape, case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda").to(torch.float32 if case["dtype"] == "f32" else torch.bfloat16)


def prepare(case, seed):
    """A pool with the weights of the tenants that the batches name, and the batches' inputs on the GPU."""
    rng = np.random.default_rng(seed + 1)
    lens0 = np.array(_lens(case), dtype=np.int32)
    r, n, d, layers = len(lens0), int(lens0.sum()), case["d"], case["layers"]
    p = _popularity(case)
    ids = [rng.choice(case["tenants"], size=r, p=p).astype(np.int32) for _ in range(case["batches"])]
    lens = [rng.permutation(lens0) for _ in range(case["batches"])]
    attention = case["block"] not in ("ffn", "adapter")
    serve = case["use"] == "serve"
    pool = hmi.Pool(block=BLOCKS[case["block"]], dtype=hmi.HMI_F32 if case["dtype"] == "f32" else hmi.HMI_BF16, d_model=d,
                    d_ff=case["ff"], n_heads=d // 64 if attention else 0, n_layers=layers, max_tenants=case["tenants"],
                    hbm_slots=min(case["slots"] or case["tenants"], case["tenants"]), host_tier=case["slots"] > 0,
                    max_requests=r, max_tokens=n, ln_eps=1e-5 if "decoder" in case["block"] else 1e-12,
                    compute_stream=torch.cuda.current_stream().cuda_stream, adapter_rank=RANK,
                    max_classes=CLASSES if serve else 0)
    draws = _Draws(case, seed)
    shared, own = _shared_shapes(case), _own_shapes(case)
    if shared:
        for layer in range(layers):
            pool.load_shared(layer, draws.tensors(shared))
    present = sorted(set(np.concatenate(ids).tolist()))
    if case["slots"]:
        # the ids share the weight sets of the first few: in HBM every id still has its own slot and its own copies
        sources = range(min(IMAGES, case["tenants"]))
        for t in sources:
            for layer in range(layers):
                pool.load_tenant(t, layer, draws.tensors(own))
        for t in range(len(sources), case["tenants"]):
            pool.alias_tenant(t, t % len(sources))
    else:
        for t in present:
            for layer in range(layers):
                pool.load_tenant(t, layer, draws.tensors(own))
    state = {"pool": pool, "case": case, "ids": ids, "lens": lens}
    if serve:
        for t in present:      # three tenants in ten tag every row, the others classify on the first
            classes = int(rng.integers(2, CLASSES + 1))
            pool.load_head(t, draws.tensor((classes, d), "w"), draws.tensor((classes,), "b"), bool(rng.random() < 0.3))
        state["table"] = _normal((TABLE, 3, d), case, seed + 2)
        state["fragments"] = torch.from_numpy(rng.integers(0, TABLE, size=n).astype(np.int32)).cuda()
        state["x"] = torch.empty((n, d), device="cuda", dtype=state["table"].dtype)
        state["scores"] = torch.empty((n, CLASSES), device="cuda", dtype=torch.float32)
        state["labels"] = torch.empty((n,), device="cuda", dtype=torch.int32)
    else:
        state["x"] = _normal((case["batches"] * n, d), case, seed + 2)
    state["y"] = torch.empty_like(state["x"])
    if case["use"] == "generate":
        pool.kv_create(r, int(lens0.max()) + case["steps"])
        state["lines"] = rng.permutation(r).astype(np.int32)
        state["tokens"] = _normal((case["steps"], r, d), case, seed + 3)
        state["made"] = torch.empty_like(state["tokens"])
    if case["use"] == "queue":
        state["queue"] = hmi.Queue(pool, r, n, max_waiting_batches=2)
        off = np.concatenate([[0], np.cumsum(np.concatenate(lens))])
        state["rows"] = [(state["x"][off[i]:off[i + 1]], state["y"][off[i]:off[i + 1]]) for i in range(len(off) - 1)]
    return state


# ---------------------------------------------------------------- one pass

def _queue_pass(state):
    queue, r = state["queue"], state["case"]["requests"]
    tickets, fetched = [], 0

    def run_one():
        nonlocal fetched
        queue.run()
        for i in range(fetched, fetched + r):
            queue.fetch(tickets[i], state["rows"][i][1])
        fetched += r

    for b, ids in enumerate(state["ids"]):
        for i in range(r):
            tickets.append(queue.push(int(ids[i]), state["rows"][b * r + i][0]))
        if b:
            run_one()           # while the next batch waits, so that its tenants are brought in under this one's kernels
    run_one()
    return state["y"]


def run(state):
    case, pool = state["case"], state["pool"]
    ids, lens = state["ids"][0], state["lens"][0]
    if case["use"] == "queue":
        return _queue_pass(state)
    if case["use"] == "generate":
        pool.prefill(0, case["layers"], state["x"], state["y"], ids, lens, state["lines"])
        for i in range(case["steps"]):
            pool.decode_step(0, case["layers"], state["tokens"][i], state["made"][i], ids, state["lines"])
        return state["y"], state["made"]
    if case["use"] == "serve":
        pool.plot_aggregate(state["table"], state["fragments"], lens, state["x"])
        pool.stack_forward(0, case["layers"], state["x"], state["y"], ids, lens)
        pool.head_forward(state["y"], state["scores"], state["labels"])
        return state["y"], state["scores"], state["labels"]
    pool.stack_forward(0, case["layers"], state["x"], state["y"], ids, lens)
    return state["y"]


def tolerance(case):
    """Four times the distance from the same path in 64 bits (24 requests of every listed case and of ten drawn ones).
    fp32, sums of up to 3072 products: 6e-7, one value 4e-6.  bf16, operands rounded between the products, hidden states of up
    to six layers carrying all of those roundings, results rounded once (half a unit is 2e-3 of a value): 2.7e-3, one value
    1.4e-2.  Labels: 3 of 9 500 rows, two classes whose scores are closer than that; one label may always change."""
    if case["dtype"] == "f32":
        return {"rel": 2.4e-6, "max": 1.6e-5}
    return {"rel": 1.1e-2, "max": 5.5e-2, "differ": max(1.3e-3, 1.001 / sum(_lens(case)))}
