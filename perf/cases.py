"""The work a serving program has this library do, as cases with sizes, inputs, tolerances and 64-bit references.

A case is one call path of the C ABI binding:
  kind "attn"    one layer's compute stage over a prefix that is resident: suffix append + paged causal GQA attention,
                 through calvo_prefill_attn ("call"), a prepared batch ("batch") or calvo_prefill_attn_noalloc ("noalloc")
  kind "ingest"  the loading stage: a prefix in pinned host memory to the paged pool, all layers, until it is resident
  kind "step"    a whole request: loading of every layer with each layer's attention queued behind it

Lengths are those of the package's workload recipes (workload.py), of the paper's Table 1 and of the tests.  A request's
lengths are written "P+S" (cached tokens, query tokens), requests separated by commas.
"""
import math
import weakref

import numpy as np
import torch

from paper_2603_21257_amd import binding as cb
from paper_2603_21257_amd import workload as wl

B = wl.BLOCK_TOKENS
TABLE1 = ",".join("%d+%d" % ps for ps in wl.TABLE1_MEAN_LENGTHS)


def _case(name, kind, lens, hq=32, hkv=8, dim=128, dtype="bf16", layers=1, entry="batch", shared=0, chunk=0):
    c = {"kind": kind, "lens": lens, "hq": hq, "hkv": hkv, "dim": dim, "dtype": dtype, "layers": layers, "entry": entry,
         "shared": shared, "chunk": chunk}
    return dict({"name": name}, **c) if name else c


def _varlen_lens():
    """The lengths of the 8-request batch recipe (requests that share a 4096-token run)."""
    _, reqs = wl.config_shape_and_requests(4)
    return ",".join("%d+%d" % (r.prefix_len, r.suffix_len) for r in reqs)


def listed():
    return [
        # smallest call: one new token behind a short cached prompt; launches and host time are what it costs
        _case("one_token_512", "attn", "512+1", entry="call"),
        # one request of the paper's regime: 28096 cached tokens, 28 query tokens (Table 1)
        _case("query28_28k", "attn", "28096+28"),
        # the three Table 1 means as one batch (ragged query lengths, long contexts)
        _case("table1_batch", "attn", TABLE1),
        # second model family (40 query heads in 8 groups of 5) with a short query over a long context
        _case("group5_query209_38k", "attn", "38304+209", hq=40, entry="call"),
        # 16K cached + 2K computed tokens, per-call entry point
        _case("prefill_16k_2k", "attn", "16384+2048", entry="call"),
        # the 64K-context workload that the headline number is quoted on
        _case("prefill_60k_4k", "attn", "61440+4096"),
        # 8 requests of 8K-32K tokens that share a 4096-token run
        _case("varlen_batch8", "attn", _varlen_lens(), shared=4096),
        # largest: one layer of the 64-query-head stack, 120K cached + 8K computed tokens
        _case("prefill_120k_8k", "attn", "122880+8192", hq=64),
        # fp32 pool, 64-wide heads: workload 1
        _case("fp32_1k_128", "attn", "1024+128", hq=8, hkv=2, dim=64, dtype="f32", entry="call"),
        # bf16 with 64-wide heads: a model family outside the 128-wide ones, ragged query
        _case("head64_4k_300", "attn", "4096+300", hq=16, hkv=4, dim=64),
        # loading stage: 16K cached tokens of a 4-layer slice of the stack
        _case("ingest_16k", "ingest", "16384+0", layers=4, entry="call"),
        # a whole request: 4K cached tokens loaded over 8 layers, a 1000-token query computed layer by layer
        _case("step_4k_1000", "step", "4096+1000", layers=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: attention at bf16 / 128 most often, then the other element types and head widths, then loading and whole
    requests.  Head layouts, lengths, batch size, shared run and entry point are drawn."""
    kind = rng.choices(["main", "other", "ingest", "step"], [6, 3, 1, 1])[0]
    entry = rng.choice(["call", "batch", "batch", "noalloc"])
    if kind == "main":
        hq, hkv = rng.choice([(32, 8), (32, 8), (40, 8), (64, 8), (16, 2), (8, 8)])
        n = rng.choice([1, 1, 1, 2, 4])
        shared = rng.choice([0, 0, 1024]) if n > 1 else 0
        lens = []
        for _ in range(n):
            # short queries over long contexts, ordinary prefills, and prefills without any cached prefix
            p = rng.choice([0, 1, 1, 1, 1, 1]) * _log_int(rng, 64, 65536) // B * B
            s = _log_int(rng, 1, 512) if rng.random() < 0.6 else _log_int(rng, 512, 4096)
            lens.append((max(p, shared), s))
        if entry == "noalloc" and (n > 1 or lens[0][1] > 64):
            entry = "call"                 # the fixed-size array of that entry point holds single short queries
        return _case(None, "attn", ",".join("%d+%d" % x for x in lens), hq, hkv, entry=entry, shared=shared)
    if kind == "other":
        dtype = rng.choice(["f32", "bf16"])
        dim = rng.choice([40, 64, 64, 80, 96, 256] if dtype == "bf16" else [40, 64, 64, 128, 256])
        hq, hkv = rng.choice([(8, 2), (16, 4), (6, 3), (8, 8), (10, 2), (32, 8)])
        n = rng.choice([1, 1, 3])
        lens = [(rng.choice([0, 1, 1, 1]) * _log_int(rng, 32, 8192) // B * B, _log_int(rng, 1, 512)) for _ in range(n)]
        return _case(None, "attn", ",".join("%d+%d" % x for x in lens), hq, hkv, dim, dtype, entry=entry)
    if kind == "ingest":
        return _case(None, "ingest", "%d+0" % (_log_int(rng, 256, 32768) // B * B), *rng.choice([(32, 8), (16, 2)]),
                     layers=rng.randint(1, 6), entry="call", chunk=rng.choice([0, 0, 64, 254]))
    return _case(None, "step", "%d+%d" % (_log_int(rng, 512, 16384) // B * B, _log_int(rng, 16, 2048)),
                 layers=rng.randint(2, 8), chunk=rng.choice([0, 0, 128]))


# ---- inputs

def _lens(case):
    return [tuple(int(x) for x in ps.split("+")) for ps in case["lens"].split(",")]


def _tdtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _workload(case, seed):
    lens = _lens(case)
    sb = case["shared"] // B
    need = sb + sum(p // B - sb + -(-s // B) for p, s in lens)
    shape = wl.Shape(case["layers"], case["hq"], case["hkv"], case["dim"], case["dtype"], need * 5 // 4 + 8)
    return wl.make_custom(shape, lens, seed, shared_blocks=sb, with_payload=False)


def _normal(shape, dtype, seed, key):
    """N(0,1) values on the GPU, rounded to the stored type."""
    return wl.fill_normal_(torch.empty(shape, dtype=dtype, device="cuda:0"), (seed << 4) + key)


class _Handles:
    """Context and prepared batch of one state; given back when the state goes."""

    def __init__(self, ctx, batch, keep):
        self.ctx, self.batch = ctx, batch
        self._fin = weakref.finalize(self, _Handles._close, ctx, batch, keep)

    @staticmethod
    def _close(ctx, batch, keep):
        if batch:
            cb.calvo_batch_destroy(batch)
        cb.calvo_destroy(ctx)
        del keep


def prepare(case, seed):
    w = _workload(case, seed)
    s, dt = w.shape, _tdtype(case)
    L, T = s.n_layers, w.total_suffix
    pool = _normal((L, s.pool_blocks, 2, B, s.n_kv_heads, s.head_dim), dt, seed, 1)
    st = {"kind": case["kind"], "entry": case["entry"], "layers": L, "pool": pool, "cu": w.cu_suffix, "w": w}
    if T:
        st["q"] = _normal((L, T, s.n_q_heads, s.head_dim), dt, seed, 2)
        st["ks"] = _normal((L, T, s.n_kv_heads, s.head_dim), dt, seed, 3)
        st["vs"] = _normal((L, T, s.n_kv_heads, s.head_dim), dt, seed, 4)
        st["out"] = torch.zeros((L, T, s.n_q_heads, s.head_dim), dtype=dt, device="cuda:0")
    loads = case["kind"] != "attn"
    host = None
    if loads:
        host = torch.empty((L, w.host_blocks, s.blk_elems), dtype=dt, pin_memory=True)
        host.copy_(_normal(host.shape, dt, seed, 5))
        st["host"] = host
        pool.zero_()                        # the loading stage writes it
    stride = w.host_blocks * s.blk_bytes
    st["reqs"] = [cb.make_request(host.data_ptr() + r.host_block_start * s.blk_bytes if loads else None, stride if loads else 0,
                                  r.table, r.n_prefix_blocks, r.suffix_len,
                                  r.first_ingest_block if loads else r.n_prefix_blocks) for r in w.requests]
    # chunk-granular loading of the last layer (its attention follows the chunks)
    st["chunks"] = [0] * (L - 1) + [case["chunk"]] if case["chunk"] else None
    torch.cuda.synchronize()
    ctx = cb.calvo_create(L, s.n_q_heads, s.n_kv_heads, s.head_dim, cb.CALVO_BF16 if case["dtype"] == "bf16" else cb.CALVO_F32,
                          s.pool_blocks, pool, staging_bytes=(128 << 20) if loads else 0)
    batch = cb.calvo_batch_prepare(ctx, st["reqs"], w.cu_suffix) if case["entry"] == "batch" and T else None
    st["h"] = _Handles(ctx, batch, [pool, host, st.get("out")])
    return st


# ---- one pass

def _load(st):
    if st["chunks"]:
        cb.calvo_kv_ingest_chunked(st["h"].ctx, st["reqs"], 0, st["layers"], st["chunks"])
    else:
        cb.calvo_kv_ingest(st["h"].ctx, st["reqs"], 0, st["layers"])


def _attn(st, l):
    a = (st["q"][l], st["ks"][l], st["vs"][l], st["out"][l])
    if st["entry"] == "batch":
        cb.calvo_prefill_attn_batch(st["h"].ctx, st["h"].batch, l, *a)
    elif st["entry"] == "noalloc":
        cb.calvo_prefill_attn_noalloc(st["h"].ctx, l, *a, st["reqs"], st["cu"])
    else:
        cb.calvo_prefill_attn(st["h"].ctx, l, *a, st["reqs"], st["cu"])


def run(st):
    if st["kind"] == "ingest":
        _load(st)
        cb.calvo_layer_event(st["h"].ctx, st["layers"] - 1, cb.CALVO_EV_HOST_WAIT)
        return {"pool": st["pool"].view(torch.int32)}
    if st["kind"] == "step":
        _load(st)
        for l in range(st["layers"]):
            _attn(st, l)
        torch.cuda.synchronize()            # the first token is out: the request is answered here
    else:
        _attn(st, 0)
    return {"out": st["out"], "pool": st["pool"]}


# ---- what a pass cannot do without, and how exact it is

def work(case):
    lens, sb = _lens(case), case["shared"]
    elt = 2 if case["dtype"] == "bf16" else 4
    kv = 2 * case["hkv"] * case["dim"] * elt
    prefix = sum(p for p, _ in lens) - sb * (len(lens) - 1)
    suffix = sum(s for _, s in lens)
    pairs = sum(s * p + s * (s + 1) // 2 for p, s in lens)
    nbytes = flops = 0
    if case["kind"] != "attn":
        nbytes += 2 * prefix * kv                                     # host read, pool write
    if case["kind"] != "ingest":
        # cached K/V read; suffix K/V read and stored; q read, out written
        nbytes += (prefix + 2 * suffix) * kv + 2 * suffix * case["hq"] * case["dim"] * elt
        flops += 4 * case["dim"] * case["hq"] * pairs
    return {"bytes": nbytes * case["layers"], "flops": flops * case["layers"]}


def tolerance(case):
    if case["kind"] == "ingest":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 1e-4}
    # bf16: output rounding (2^-9 at most) and weights rounded to bf16 before the second product
    return {"rel": 1e-2, "max": 5e-2}


def exact(case, seed):
    """Textbook attention in 64 bits on the stored inputs; nothing for bytes that are only moved."""
    if case["kind"] == "ingest":
        return None
    w = _workload(case, seed)
    s, dt = w.shape, _tdtype(case)
    L, T, D = s.n_layers, w.total_suffix, s.head_dim
    q, ks, vs = (_normal((L, T, h, D), dt, seed, k) for h, k in ((s.n_q_heads, 2), (s.n_kv_heads, 3), (s.n_kv_heads, 4)))
    if case["kind"] == "attn":
        pool, host = _normal((L, s.pool_blocks, 2, B, s.n_kv_heads, D), dt, seed, 1), None
    else:
        pool, host = None, _normal((L, w.host_blocks, s.blk_elems), dt, seed, 5).view(L, w.host_blocks, 2, B, s.n_kv_heads, D)
    scale = float(np.float32(1.0) / np.sqrt(np.float32(D)))
    out = torch.empty((L, T, s.n_q_heads, D), dtype=torch.float64, device="cuda:0")
    group = s.n_q_heads // s.n_kv_heads
    for l in range(L):
        for r, a in zip(w.requests, w.cu_suffix):
            a, P, S = int(a), r.prefix_len, r.suffix_len
            if S == 0:
                continue
            if host is None:
                blocks = pool[l][torch.from_numpy(r.table[:r.n_prefix_blocks].astype(np.int64)).to("cuda:0")]
            else:
                blocks = host[l, r.host_block_start:r.host_block_start + r.n_prefix_blocks]
            for g in range(s.n_kv_heads):
                k = torch.cat([blocks[:, 0, :, g].reshape(P, D), ks[l, a:a + S, g]]).double()
                v = torch.cat([blocks[:, 1, :, g].reshape(P, D), vs[l, a:a + S, g]]).double()
                kt = k.t().contiguous()
                rows = max(1, min(S, (1 << 27) // (P + S)))
                for i in range(0, S, rows):
                    n = min(rows, S - i)
                    seen = torch.arange(P + S, device="cuda:0")[None, :] <= P + i + torch.arange(n, device="cuda:0")[:, None]
                    for h in range(g * group, (g + 1) * group):
                        x = torch.matmul(q[l, a + i:a + i + n, h].double(), kt)
                        x.mul_(scale).masked_fill_(~seen, -math.inf)
                        out[l, a + i:a + i + n, h] = torch.matmul(torch.softmax(x, dim=1), v)
    return {"out": out, "pool": None}
