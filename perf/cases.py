"""The work whose time is watched: packs, snapshots, restores and verifies of one rank's training state.

A case names an operation, the state's layout and the mode of the context:

  op      pack      ckpt_pack_noalloc: fragments -> the caller's device image and its chunk sums
          snapshot  Checkpointer.snapshot, the gate before the optimizer step, the wait for the commit
          restore   Checkpointer.restore of a committed image into live tensors that hold something else
          verify    Checkpointer.verify of a committed image
  layout  gpt       the parameters of a GPT, each with its fp32 master copy and Adam moments (14 bytes a
                    parameter), registered parameter by parameter; every fragment aligned as an allocator would
          llama     the same for LLaMA layers under tensor parallelism, without embedding and head
          ragged    `frags` tensors of log-uniform sizes, bf16 and fp32 in turn, `bytes` in all, each aligned
          views     the same sizes back to back in two flat buffers, as a distributed optimizer hands out its
                    shards: aligned to their element only
  mode    staged    full device image (the default); ring: a staging ring; direct: no device image, the DMA
                    engines gather; bounce: pageable host images behind pinned rings

The library moves bytes and adds 64-bit words modulo 2^64, so every output is exact.
"""
import random

import numpy as np
import torch

import paper_2607_01646_amd as P

KiB, MiB, GiB = 1 << 10, 1 << 20, 1 << 30

GPT_1L_H64 = dict(layout="gpt", layers=1, hidden=64, ffn=256, vocab=256, seq=64)
GPT_4L_H512 = dict(layout="gpt", layers=4, hidden=512, ffn=2048, vocab=8192, seq=512)
GPT_8L_H1024 = dict(layout="gpt", layers=8, hidden=1024, ffn=4096, vocab=8192, seq=1024)
LLAMA_RANK = dict(layout="llama", layers=10, hidden=8192, ffn=22016, tp=8)


def listed():
    return [
        # The smallest call: the state of a toy model (1 MB, 64 fragments), packed inside a loop that may not
        # allocate. Its time is launches and host work.
        dict(name="pack-small", op="pack", chunk=64 * KiB, **GPT_1L_H64),
        # An ordinary small shard (239 MB, 208 fragments, 4 MiB chunks).
        dict(name="pack-gpt", op="pack", chunk=4 * MiB, **GPT_4L_H512),
        # One rank of a 65B model under TP=8 x PP=8 (14.2 GB, 360 fragments): the HBM-bound end of the range.
        dict(name="pack-llama-rank", op="pack", chunk=64 * MiB, **LLAMA_RANK),
        # Many tensors of every size (4096 fragments, 8 GiB).
        dict(name="pack-ragged", op="pack", layout="ragged", frags=4096, bytes=8 * GiB, chunk=64 * MiB),
        # A distributed optimizer's flat buffers: fragments start and end anywhere (512 of them, 1 GiB).
        dict(name="pack-views", op="pack", layout="views", frags=512, bytes=1 * GiB, chunk=16 * MiB),
        # A snapshot of a state so small that latency is all of it.
        dict(name="snapshot-small", op="snapshot", mode="staged", chunk=64 * KiB, **GPT_1L_H64),
        # A snapshot of the ordinary small shard, in the default mode.
        dict(name="snapshot-gpt", op="snapshot", mode="staged", chunk=4 * MiB, **GPT_4L_H512),
        # The mode for long compute windows: nothing staged on the device (1.5 GB, 400 fragments).
        dict(name="snapshot-direct", op="snapshot", mode="direct", chunk=64 * MiB, **GPT_8L_H1024),
        # The mode for states larger than the pinned memory the host grants: pageable images.
        dict(name="snapshot-bounce", op="snapshot", mode="bounce", chunk=16 * MiB, **GPT_4L_H512),
        # Recovery of the small shard from its own host image.
        dict(name="restore-gpt", op="restore", mode="staged", chunk=4 * MiB, **GPT_4L_H512),
        # Recovery into a distributed optimizer's flat buffers.
        dict(name="restore-views", op="restore", mode="staged", layout="views", frags=1024, bytes=512 * MiB,
             chunk=16 * MiB),
        # The integrity check of a committed snapshot.
        dict(name="verify-gpt", op="verify", mode="staged", chunk=4 * MiB, **GPT_4L_H512),
    ]


def _log_between(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng: random.Random):
    op = rng.choice(["pack", "pack", "pack", "snapshot", "snapshot", "restore", "verify"])
    c = dict(op=op)
    if rng.random() < 0.4:
        hidden = 8 * _log_between(rng, 8, 128 if op != "pack" else 256)
        c.update(layout="gpt", layers=rng.randint(1, 8), hidden=hidden, ffn=4 * hidden - 8 * rng.randint(0, 3),
                 vocab=_log_between(rng, 200, 8192), seq=_log_between(rng, 64, 1024))
    else:
        frags = _log_between(rng, 1, 4096 if op == "pack" else 1024)
        size = _log_between(rng, max(256 * KiB, 256 * frags), 4 * GiB if op == "pack" else 768 * MiB)
        c.update(layout=rng.choice(["ragged", "views"]), frags=frags, bytes=size)
    # Chunks of 64 KiB to 64 MiB, one in four of them no power of two, at most 4096 chunks in all.
    unit = rng.choice([1, 1, 1, 3])
    lo = 64 * KiB
    while unit * lo * 4096 < _payload(c):
        lo *= 2
    c["chunk"] = unit * lo * 2 ** rng.randint(0, max(0, (64 * MiB // (unit * lo)).bit_length() - 1))
    c["align"] = rng.choice([256, 256, 256, 64, 512, 4096])
    if op != "pack":
        c["mode"] = rng.choice(["staged", "staged", "ring", "direct", "bounce"])
    return c


# ---- layouts ----


def _param_counts(case):
    h, f = case["hidden"], case["ffn"]
    if case["layout"] == "gpt":
        layer = [h, h, 3 * h * h, 3 * h, h * h, h, h, h, f * h, f, h * f, h]
        return [case["vocab"] * h, case["seq"] * h] + layer * case["layers"] + [h, h]
    tp = case["tp"]
    return [h, h // tp * h, h // tp * h, h // tp * h, h * h // tp, h, f // tp * h, f // tp * h,
            h * (f // tp)] * case["layers"]


def _sizes(case):
    """[(flat buffer, bytes)] in registration order; the buffers are of the element sizes _ELEMENTS gives."""
    if case["layout"] in ("gpt", "llama"):
        out = []
        for n in _param_counts(case):
            out += [(0, 2 * n), (1, 4 * n), (2, 4 * n), (3, 4 * n)]
        return out
    n, total = case["frags"], case["bytes"]
    r = np.random.Generator(np.random.PCG64(n * 1000003 + total))  # the layout belongs to the case, not to the seed
    raw = np.exp(r.uniform(np.log(1024.0), np.log(float(64 * MiB)), n))
    raw *= total / raw.sum()
    return [(k % 2, max(1, int(x) // e) * e) for k, x in enumerate(raw) for e in (2 + 2 * (k % 2),)]


def _dtypes(case):
    return [torch.bfloat16] + [torch.float32] * (3 if case["layout"] in ("gpt", "llama") else 1)


def _payload(case):
    return sum(n for _, n in _sizes(case))


def _align(case):
    return case.get("align", 256)


def _image(case):
    """Image offsets of the fragments and the image's size, by the layout's definition."""
    a, end, off = _align(case), 0, []
    for _, n in _sizes(case):
        off.append(-(-end // a) * a)
        end = off[-1] + n
    return off, -(-end // a) * a


def _fragments(case, seed):
    """The flat buffers, filled from the seed, and the fragments in them."""
    step = 1 if case["layout"] == "views" else 512  # bytes a fragment's start is a multiple of (torch's allocator: 512)
    dts = _dtypes(case)
    used, at = [0] * len(dts), []
    for b, n in _sizes(case):
        at.append((b, used[b], n))
        used[b] = -(-(used[b] + n) // step) * step
    g = torch.Generator(device="cuda").manual_seed(seed)
    flat = []
    for k, dt in enumerate(dts):
        t = torch.empty(-(-used[k] // 8) * 8 // dt.itemsize, dtype=dt, device="cuda")
        t.normal_(0.0, 0.02 if k < 2 else 1e-3, generator=g)  # parameters and master copies, then the moments
        flat.append(t.mul_(t) if k == 3 else t)
    frags = [flat[b][o // dts[b].itemsize:(o + n) // dts[b].itemsize] for b, o, n in at]
    return flat, frags


# ---- one pass ----


class _Kept(np.ndarray):
    """A borrowed view of a context's host memory that keeps the context alive."""


def _kept(a, owner):
    v = a.view(_Kept)
    v.owner = owner
    return v


def prepare(case, seed):
    flat, frags = _fragments(case, seed)
    st = dict(case=case, flat=flat, frags=frags, step=0)
    if case["op"] == "pack":
        off, image, chunks = P.ckpt_plan([n for _, n in _sizes(case)], case["chunk"], _align(case))
        st["image"] = torch.empty(image, dtype=torch.uint8, device="cuda")
        st["sums"] = torch.empty(chunks, dtype=torch.int64, device="cuda")
        return st
    chunk = case["chunk"]
    mode = case["mode"]
    opts = {}
    if mode == "ring":  # a quarter of the image, four slots
        opts["device_staging_bytes"] = max(4, _image(case)[1] // (4 * chunk)) * chunk
    elif mode == "direct":
        opts["direct"] = True
    elif mode == "bounce":  # DMA groups of 64 MiB in rings of four
        group = max(chunk, 64 * MiB // chunk * chunk)
        opts.update(group_bytes=group, bounce_bytes=4 * group)
    st["ck"] = P.Checkpointer(frags, chunk_bytes=chunk, align_bytes=_align(case), **opts)
    if case["op"] != "snapshot":
        torch.cuda.synchronize()
        st["ck"].wait_committed(st["ck"].snapshot(step=1, meta=b"rng"))
        for t in flat:  # the live tensors are lost
            t.zero_()
        torch.cuda.synchronize()
    return st


def run(st):
    op = st["case"]["op"]
    if op == "pack":
        P.ckpt_pack_noalloc(st["frags"], st["image"], st["sums"], st["case"]["chunk"], _align(st["case"]))
        return {"image": st["image"], "sums": st["sums"]}
    ck = st["ck"]
    if op == "snapshot":
        st["step"] += 1
        snap = ck.snapshot(step=st["step"], meta=b"rng")
        ck.wait_captured(snap)
        ck.wait_committed(snap)
        image, sums = ck.host_image(snap)
        return {"image": _kept(image, ck), "sums": _kept(sums, ck).view(np.int64)}
    if op == "restore":
        bad = ck.restore()
        return {"flat": [t.view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32) for t in st["flat"]],
                "bad": len(bad)}
    bad = ck.verify()
    return {"sums": P.ckpt_last_sums(ck.ctx).view(np.int64), "bad": len(bad)}


def work(case):
    payload, image = _payload(case), _image(case)[1]
    sums = 8 * -(-image // case["chunk"])
    if case["op"] == "verify":
        return {"bytes": image + sums, "flops": 0}
    return {"bytes": payload + image + sums, "flops": 0}


def tolerance(case):
    return "exact"


def exact(case, seed):
    """What run() returns, from torch copies and 64-bit sums alone."""
    if _image(case)[1] > 2 * GiB:
        return None
    flat, frags = _fragments(case, seed)
    if case["op"] == "restore":
        return {"flat": [t.view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32) for t in flat], "bad": 0}
    off, size = _image(case)
    image = torch.zeros(size, dtype=torch.uint8, device="cuda")
    for o, t in zip(off, frags):
        b = t.view(torch.uint8)
        image[o:o + b.numel()] = b
    sums = torch.stack([image[lo:lo + case["chunk"]].view(torch.int64).sum() for lo in range(0, size, case["chunk"])])
    if case["op"] == "verify":
        return {"sums": sums.cpu().numpy(), "bad": 0}
    if case["op"] == "snapshot":
        return {"image": image.cpu().numpy(), "sums": sums.cpu().numpy()}
    return {"image": image, "sums": sums}
