"""What a user of this library has it do, as measurable cases: one node's share of a gradient exchange, through the
functions of paper_2310_06993_amd.binding.

A case is one call (two with the transform switched off) on tensors that are already on the GPU.  Its `op`:

  fused          or_fused_path / _bf16            raw slices of N workers -> decoded mean of one shard, counts
  fused_batched  or_fused_path_batched_monitored  the same for all DDP buckets of a gradient, with the loss totals
  encode         or_rht_encode_at / _bf16         a worker encodes its own gradient before it is cut into shards
  reduce_decode  or_reduce_decode / _bf16         encoded shards of N workers -> decoded mean, counts
  decode         or_rht_decode_masked / _bf16     a worker decodes the aggregated gradient after a lossy broadcast
  transform_off  or_masked_reduce + or_finalize   aggregation at losses too low for the transform to be switched on

Inputs come from paper_2310_06993_amd.workloads (its value and drop recipes).  Inputs that stand for encoded data are
Gaussian, which is what the transform makes of a gradient.
"""
from __future__ import annotations

import math

import torch

import paper_2310_06993_amd.binding as b
from paper_2310_06993_amd import workloads as wl

SHARD = 1   # which shard this node owns (worker 1's own slice always arrives)
MIB = 1 << 20


def _case(op, dtype, workers, entries, k, name=None, values="normal", drops="iid_packet", loss=0.01, packet=256, burst=8.0,
          bucket=0):
    """`entries`: of one worker's gradient.  encode and decode work on all of it, the other ops on one shard of it
    (padded to whole blocks).  `bucket`: entries of one bucket (fused_batched)."""
    c = {"op": op, "dtype": dtype, "workers": workers, "entries": entries, "k": k, "values": values, "drops": drops,
         "loss": loss, "packet": packet, "burst": burst, "bucket": bucket}
    return {"name": name, **c} if name else c


def listed():
    tiny, r50, bert, gpt2, llama = (wl.CONFIGS[n] for n in wl.ORDER)
    return [
        # a very small gradient: the call and the launch are all there is
        _case("fused", "f32", 4, tiny.entries, 10, "tiny_fused", drops="iid_entry"),
        # one 25 MiB DDP bucket of bf16 gradients at a worker, as the backward pass hands it over
        _case("encode", "bf16", 16, 25 * MIB // 2, 12, "bucket_encode_bf16"),
        # one 25 MiB DDP bucket at the node that owns a shard of it, aggregated as soon as it is there
        _case("fused", "f32", 16, gpt2.bucket_entries, 12, "bucket_fused", loss=0.05),
        # a ResNet-50-sized gradient in one call; 1 % of the entries are outliers
        _case("fused", "f32", 8, r50.entries, 12, "resnet50_fused", values="outliers"),
        # the same gradient back at a worker; its length is no multiple of the block
        _case("decode", "f32", 8, r50.entries, 12, "resnet50_decode"),
        # the same in bf16 on a quiet network: sum, count and mean without the transform
        _case("transform_off", "bf16", 8, r50.entries, 12, "resnet50_transform_off_bf16", loss=0.001),
        # a BERT-large-sized gradient: layers of very different scale, bursts of lost packets
        _case("fused", "f32", 8, bert.entries, 14, "bert_large_fused", values="layers", drops="gilbert", loss=0.02),
        # the same from mixed-precision training
        _case("fused", "bf16", 8, bert.entries, 14, "bert_large_fused_bf16", values="layers", drops="gilbert", loss=0.02),
        # the same shard where the workers encoded before they sent
        _case("reduce_decode", "f32", 8, bert.entries, 14, "bert_large_reduce_decode", drops="gilbert", loss=0.02),
        # all 238 buckets of a GPT-2-XL-sized gradient in one call, with the loss totals
        _case("fused_batched", "f32", 16, gpt2.entries, 12, "gpt2_xl_fused_batched", loss=0.05, bucket=gpt2.bucket_entries),
        # a Llama-8B-sized gradient: the longest shard, the largest blocks
        _case("fused", "bf16", 8, llama.entries, 16, "llama_8b_fused_bf16", drops="gilbert", packet=512, burst=32.0),
        # the same gradient at a worker, encoded in eight parts while the backward pass goes on: one part
        _case("encode", "bf16", 8, llama.entries // 8, 16, "llama_8b_encode_bf16"),
    ]


def draw(rng):
    """Any op, either type, blocks of 2^8 .. 2^16, 2 .. 32 workers, 256 KiB .. 2 GiB of input, odd lengths."""
    op = rng.choice(("fused", "fused", "fused_batched", "encode", "reduce_decode", "decode", "transform_off"))
    dtype = rng.choice(("f32", "bf16"))
    es = 4 if dtype == "f32" else 2
    k = rng.randint(8, 16)
    workers = rng.choice((2, 3, 4, 5, 6, 8, 8, 12, 16, 24, 32))
    size = math.exp(rng.uniform(math.log(MIB / 4), math.log(2048 * MIB)))
    entries = int(size / es) | 1
    bucket = 0
    drops = rng.choice(("iid_packet", "gilbert", "iid_entry" if entries < 1 << 25 else "gilbert"))
    if op == "fused_batched":
        drops = "iid_packet"
        bucket = max(rng.choice((25, 4)) * MIB // es, entries // 256)
    return _case(op, dtype, workers, entries, k, values=rng.choice(("normal", "outliers", "layers")), drops=drops,
                 loss=round(math.exp(rng.uniform(math.log(1e-3), math.log(5e-2))), 5), packet=rng.choice((256, 512)),
                 burst=rng.choice((4.0, 8.0, 32.0)), bucket=bucket)


def _config(case, seed, **changes):
    kw = dict(name=case["op"], workers=case["workers"], dtype=case["dtype"], entries=case["entries"], block_log2=case["k"],
              sigma=1.0 if case["values"] == "layers" else 1e-3, values=case["values"], drops=case["drops"],
              loss=case["loss"], packet=case["packet"], burst=case["burst"], bucket_entries=case["bucket"], seed=seed)
    kw.update(changes)
    return wl.Config(**kw)


def _workspace(shard_len, k):
    n = b.or_workspace_bytes(shard_len, k)
    return torch.empty(n, dtype=torch.uint8, device="cuda") if n else None


def prepare(case, seed):
    op, k, N, n = case["op"], case["k"], case["workers"], case["entries"]
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    s = {"op": op, "f32": dt == torch.float32, "k": k, "N": N, "n": n, "seed": seed + 1}
    encoded = {"values": "normal", "sigma": 1e-3}

    def empty(count, dtype):
        return torch.empty(count, dtype=dtype, device="cuda")

    if op == "encode":
        s["grad"] = wl.make_grads(_config(case, seed, workers=1), "cuda").view(-1)[:n]
        s["out"] = empty(b.or_padded_len(n, k), dt)
    elif op == "decode":
        # the aggregate is fp32 whatever the gradient's type; every entry has one sender, so one row of received bits
        s["agg"] = wl.make_grads(_config(case, seed, workers=1, dtype="f32", **encoded), "cuda").view(-1)
        s["mask"] = wl.make_masks(_config(case, seed, workers=2, entries=2 * s["agg"].numel()), "cuda")[1].contiguous()
        s["out"] = empty(n, dt)
    elif op == "fused_batched":
        cfg = _config(case, seed)
        parts = cfg.buckets()
        lens = [cfg.shard_len(size) for _, size in parts]
        s["out"], s["count"] = empty(sum(lens), dt), empty(sum(lens), torch.uint8)
        s["totals"], s["n_buckets"] = empty(len(parts), torch.int64), len(parts)
        items, at = [], 0
        for j, ((first, size), L) in enumerate(zip(parts, lens)):
            own = _config(case, seed * 1009 + j)
            items.append((wl.make_grads(own, "cuda", SHARD, size, first), wl.make_masks(own, "cuda", SHARD, size),
                          s["out"][at:at + L], s["count"][at:at + L], L, seed + 1 + j, SHARD * L))
            at += L
        s["items"], s["buckets"] = items, b.make_buckets(items)
        s["workspace"] = _workspace(max(lens), k)
    else:
        cfg = _config(case, seed, **({} if op == "fused" else encoded))
        L = s["L"] = cfg.shard_len()
        s["slices"], s["masks"] = wl.make_grads(cfg, "cuda", SHARD), wl.make_masks(cfg, "cuda", SHARD)
        s["out"], s["count"] = empty(L, dt), empty(L, torch.uint8)
        if op == "transform_off":
            s["sum"] = empty(L, torch.float32)
        else:
            s["workspace"] = _workspace(L, k)
    return s


def run(s):
    op, f32, k, N, seed, out = s["op"], s["f32"], s["k"], s["N"], s["seed"], s["out"]
    if op == "encode":
        (b.or_rht_encode_at if f32 else b.or_rht_encode_bf16)(s["grad"], s["n"], k, seed, 0, out)
        return out
    if op == "decode":
        (b.or_rht_decode_masked if f32 else b.or_rht_decode_masked_bf16)(s["agg"], s["mask"], s["n"], k, seed, 0, out)
        return out
    if op == "fused_batched":
        b.or_fused_path_batched_monitored(s["buckets"], s["n_buckets"], N, k, not f32, s["totals"], s["workspace"])
        return out, s["count"], s["totals"]
    L = s["L"]
    if op == "transform_off":
        (b.or_masked_reduce if f32 else b.or_masked_reduce_bf16)(s["slices"], s["masks"], N, L, s["sum"], s["count"])
        (b.or_finalize if f32 else b.or_finalize_bf16)(s["sum"], s["count"], L, out)
        return out, s["sum"], s["count"]
    if op == "fused":
        call = b.or_fused_path if f32 else b.or_fused_path_bf16
    else:
        call = b.or_reduce_decode if f32 else b.or_reduce_decode_bf16
    call(s["slices"], s["masks"], N, L, k, seed, SHARD * L, out, s["count"], s["workspace"])
    return out, s["count"]


def work(case):
    """Every input read once, every output written once; additions of the transforms (k per entry) and the sums."""
    op, k, N, n = case["op"], case["k"], case["workers"], case["entries"]
    es = 4 if case["dtype"] == "f32" else 2
    if op in ("encode", "decode"):
        n_pad = (n + (1 << k) - 1) >> k << k
        return {"bytes": es * (n + n_pad) if op == "encode" else 4 * n_pad + n_pad // 8 + es * n, "flops": k * n_pad}
    cfg = _config(case, 0)
    lens = [cfg.shard_len(size) for _, size in cfg.buckets()]
    L = sum(lens)
    w = {"bytes": wl.bytes_fused(N, L, es), "flops": N * L}
    if op == "transform_off":
        w["bytes"] += 4 * L
    else:
        w["flops"] += k * L * (N + 1 if op in ("fused", "fused_batched") else 1)
    if op == "fused_batched":
        w["bytes"] += 8 * len(lens)
    return w


def tolerance(case):
    """fp32: what two fp32 transforms of up to 2^16 entries differ by; bf16: results rounded to 8 bits.  The received
    counts and totals are whole numbers and agree exactly."""
    return {"rel": 2e-6} if case["dtype"] == "f32" else {"rel": 1e-2}
