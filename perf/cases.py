"""The work that a serving process has this library do, as cases to be timed.

A case is one batch of `pred` calls (or one file operation that moves K/V rows) through the public
binding, on files that are already there, as an inference scheduler issues it.  File lengths come
from the case itself ("lens": seed of the length generator), values from the seed given to
prepare().  A pass leaves the files as long as it found them (kv_truncate, kv_remove: host-side
calls that a program with draft tokens or forked branches makes anyway), so it can be repeated.

Kinds of cases
  decode   `lips` files of U{lo..hi} tokens, `new` tokens each (1 = a decode step, 2..8 = a draft being
           verified), through `layers` attention layers (1 = pred_batch; more = pred_begin / pred_layer).
           scatter: pages of a file in random places of a pool twice as large
  prompt   `lips` files of U{lo..hi} tokens (lo = hi = 0: new files), U{new_lo..new_hi} new tokens
           each: prompts and chunks of prompts
  mixed    `lips` chunks of `chunk` tokens on U{0..pre_hi} tokens, and `dec` decode files of U{lo..hi} tokens
  fork     `roots` prefixes of `prefix` tokens, each forked into `children` files with U{1..suffix} tokens
           of their own, one new token per child
  beam     the same, but the children are forked in the call, get one token and are removed again:
           a search step whose new token copies the shared, partly filled last page
  prune    kv_extract of about half of the tokens of `lips` files of U{lo..hi} tokens
  append   kv_append of U{new_lo..new_hi} tokens to each of `lips` files of U{lo..hi} tokens
"""
import random

import numpy as np
import torch

from paper_2510_25412_amd import driver, synth

P = 16          # tokens per page


def listed():
    return [
        # The smallest call: four short fp32 files, one token each; launches and host work are all there is.
        dict(name="decode_f32_tiny", kind="decode", dtype="f32", hq=8, hkv=8, lips=4, lo=37, hi=200, new=1, layers=1, scatter=False, lens=1),
        # Prompts in fp32 storage on the same head shape: four new files.
        dict(name="prompt_f32", kind="prompt", dtype="f32", hq=8, hkv=8, lips=4, lo=0, hi=0, new_lo=64, new_hi=512, lens=2),
        # One user's decode step through the attention layers of an 8B-shaped model.
        dict(name="decode_1x32_layers", kind="decode", dtype="bf16", hq=32, hkv=8, lips=1, lo=1500, hi=2500, new=1, layers=32, scatter=False, lens=3),
        # The decode batch of a loaded server: 64 files of 512..4096 tokens.
        dict(name="decode_64x8_layers", kind="decode", dtype="bf16", hq=32, hkv=8, lips=64, lo=512, hi=4096, new=1, layers=8, scatter=False, lens=4),
        # Many short conversations, in one call each.
        dict(name="decode_256_short", kind="decode", dtype="bf16", hq=32, hkv=8, lips=256, lo=100, hi=260, new=1, layers=1, scatter=False, lens=5),
        # Drafts of four tokens verified for the decode batch.
        dict(name="draft_64x4", kind="decode", dtype="bf16", hq=32, hkv=8, lips=64, lo=512, hi=4096, new=4, layers=1, scatter=False, lens=6),
        # Long contexts on a 70B-shaped layer, pages scattered.
        dict(name="decode_long_g8", kind="decode", dtype="bf16", hq=64, hkv=8, lips=16, lo=32768, hi=131072, new=1, layers=1, scatter=True, lens=7),
        # Tree search: 16 prefixes of 2048 tokens forked into 16 files each.
        dict(name="fork_tree_16x16", kind="fork", dtype="bf16", hq=32, hkv=8, roots=16, children=16, prefix=2048, suffix=256, lens=8),
        # A few users' prompts, ragged, the last chunk of each on what is there already.
        dict(name="prompt_ragged_3", kind="prompt", dtype="bf16", hq=32, hkv=8, lips=3, lo=200, hi=4000, new_lo=100, new_hi=700, lens=9),
        # A server's full batch: 32 prompt chunks of 512 tokens beside 224 decode steps.
        dict(name="mixed_32x512_224", kind="mixed", dtype="bf16", hq=32, hkv=8, lips=32, chunk=512, pre_hi=8192, dec=224, lo=1024, hi=4096, lens=10),
        # A context pruned: about half of the tokens of 64 files go to new files.
        dict(name="prune_64", kind="prune", dtype="bf16", hq=32, hkv=8, lips=64, lo=512, hi=4096, lens=11),
        # A document's K/V rows stored from elsewhere, without attention.
        dict(name="append_doc", kind="append", dtype="bf16", hq=32, hkv=8, lips=1, lo=0, hi=0, new_lo=6000, new_hi=9000, lens=12),
    ]


def _log(rng, lo, hi):
    """A whole number of lo..hi, evenly spread over its logarithm."""
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "draft", "long", "f32", "prompt", "prompt", "mixed", "fork", "beam", "prune", "append"])
    c = dict(dtype="bf16", lens=rng.randrange(1, 1 << 30))
    hkv = rng.choice([1, 2, 4, 8, 8])
    c.update(hq=hkv * rng.choice([1, 2, 4, 4, 8]), hkv=hkv)
    if kind in ("decode", "draft"):
        lo = _log(rng, 1, 2048)
        c.update(kind="decode", lips=_log(rng, 1, 256), lo=lo, hi=lo + _log(rng, 1, 2 * lo + 64), new=1 if kind == "decode" else rng.randint(2, 8),
                 layers=rng.choice([1, 1, 2, 8]), scatter=rng.random() < 0.3)
    elif kind == "long":
        lo = _log(rng, 16384, 65536)
        c.update(kind="decode", lips=_log(rng, 1, 16), lo=lo, hi=2 * lo, new=1, layers=1, scatter=True)
    elif kind == "f32":
        n, lo = rng.choice([0, 1]), _log(rng, 16, 1024)
        c.update(dtype="f32", lips=_log(rng, 1, 32))
        if n:
            c.update(kind="decode", lo=lo, hi=2 * lo, new=rng.choice([1, 1, 3]), layers=1, scatter=False)
        else:
            c.update(kind="prompt", lips=_log(rng, 1, 8), lo=0, hi=rng.choice([0, lo]), new_lo=16, new_hi=_log(rng, 32, 512))
    elif kind == "prompt":
        new = _log(rng, 16, 1024)
        c.update(kind="prompt", lips=_log(rng, 1, 16), lo=0, hi=rng.choice([0, _log(rng, 64, 8192)]), new_lo=new, new_hi=new + _log(rng, 1, new + 16))
    elif kind == "mixed":
        lo = _log(rng, 64, 2048)
        c.update(kind="mixed", lips=_log(rng, 1, 24), chunk=_log(rng, 32, 512), pre_hi=_log(rng, 64, 8192), dec=_log(rng, 1, 224), lo=lo, hi=2 * lo)
    elif kind == "fork":
        c.update(kind="fork", roots=_log(rng, 1, 16), children=_log(rng, 2, 24), prefix=_log(rng, 64, 4096), suffix=_log(rng, 1, 256))
    elif kind == "beam":
        c.update(kind="beam", roots=_log(rng, 1, 32), children=_log(rng, 2, 8), prefix=_log(rng, 64, 4096), suffix=0)
    elif kind == "prune":
        lo = _log(rng, 64, 2048)
        c.update(kind="prune", lips=_log(rng, 1, 64), lo=lo, hi=2 * lo)
    else:
        new = _log(rng, 64, 8192)
        c.update(kind="append", lips=_log(rng, 1, 4), lo=0, hi=rng.choice([0, 1000]), new_lo=new, new_hi=2 * new)
    return c


# ---- what a case consists of ------------------------------------------------------------------

def _layout(case):
    """Files [(length, root index or None, own tokens)], the batch [(file, new tokens)]."""
    r = random.Random(case["lens"])
    uni = lambda a, b: r.randint(min(a, b), max(a, b))  # noqa: E731
    kind, files, batch = case["kind"], [], []
    if kind in ("decode", "prune"):
        files = [(uni(case["lo"], case["hi"]), None) for _ in range(case["lips"])]
        batch = [(i, case.get("new", 0)) for i in range(len(files))]
    elif kind in ("prompt", "append"):
        files = [(uni(case["lo"], case["hi"]), None) for _ in range(case["lips"])]
        batch = [(i, uni(case["new_lo"], case["new_hi"])) for i in range(len(files))]
    elif kind == "mixed":
        files = [(uni(0, case["pre_hi"]), None) for _ in range(case["lips"])] + [(uni(case["lo"], case["hi"]), None) for _ in range(case["dec"])]
        batch = [(i, case["chunk"] if i < case["lips"] else 1) for i in range(len(files))]
    else:                                        # fork, beam
        for _ in range(case["roots"]):
            root = len(files)
            files.append((case["prefix"], None))
            for _ in range(case["children"]):
                batch.append((len(files), 1))
                files.append((case["prefix"] + (uni(1, case["suffix"]) if kind == "fork" else 0), root))
    return files, batch


def _shape(case):
    return synth.Shape(case["hq"], case["hkv"], 128 if case["dtype"] == "bf16" else 64, P, case["dtype"])


def _inputs(case, seed):
    """K and V rows of every file [layers, tokens, Hkv, D] (a fork's own rows only), the batch's q [layers, T, Hq, D]
    and new rows [layers, T, Hkv, D]: N(0, 1) in the storage type."""
    files, batch = _layout(case)
    s, layers = _shape(case), case.get("layers", 1)
    g = torch.Generator(device="cuda").manual_seed(seed)
    normal = lambda n, h: torch.randn((layers, n, h, s.head_dim), generator=g, device="cuda", dtype=torch.bfloat16 if s.dtype == "bf16" else torch.float32)  # noqa: E731
    own = [n - (files[root][0] if root is not None else 0) for n, root in files]
    K, V = normal(sum(own), s.n_kv_heads), normal(sum(own), s.n_kv_heads)
    T = sum(n for _, n in batch)
    return files, batch, own, K, V, normal(T, s.n_q_heads), normal(T, s.n_kv_heads), normal(T, s.n_kv_heads)


def prepare(case, seed):
    files, batch, own, K, V, q, k_new, v_new = _inputs(case, seed)
    s, kind, layers = _shape(case), case["kind"], case.get("layers", 1)
    pages = sum(-(-n // P) + 2 for n in own) + sum(-(-n // P) + 1 for _, n in batch) + (sum(-(-n // P) for n, _ in files) if kind == "prune" else 0)
    order = None
    if case.get("scatter"):
        pages *= 2
        order = np.random.Generator(np.random.PCG64(case["lens"])).permutation(pages).astype(np.int32)
    sess = driver.HipSession(s, pages, order, "cuda:0", max_lips=max(len(batch), 1), max_tokens=max(sum(n for _, n in batch), 64),
                             max_entries=sum(-(-(files[f][0] + n) // P) + 1 for f, n in batch) + 64, n_layers=layers)
    sess.pool.zero_()
    ctx, at, h = sess.ctx, 0, []
    for (n, root), m in zip(files, own):
        h.append(ctx.kv_open(None) if root is None else (ctx.kv_fork(h[root]) if kind != "beam" else -1))
        if m:
            ctx.kv_append(h[-1], m, K[:, at:at + m].contiguous(), V[:, at:at + m].contiguous(), sess.stream)
        at += m
    st = dict(kind=kind, layers=layers, sess=sess, ctx=ctx, pool=sess.pool.view(torch.int64), q=q, k=k_new, v=v_new,
              kv=np.array([h[f] for f, _ in batch], np.int32), n=np.array([n for _, n in batch], np.int32),
              lens=np.array([files[f][0] for f, _ in batch], np.int64))
    if kind == "prune":
        r = np.random.Generator(np.random.PCG64(seed))
        idx = [np.flatnonzero((np.arange(n) < P) | (r.random(n) < 0.5)) for n, _ in files]      # the first page is kept (shared)
        st["off"] = np.concatenate([[0], np.cumsum([len(i) for i in idx])]).astype(np.int64)
        st["idx"] = np.concatenate(idx).astype(np.int64)
    elif kind == "append":
        ends = np.cumsum([n for _, n in batch]).tolist()
        st["parts"] = [(int(st["kv"][i]), n, k_new[:, e - n:e].contiguous(), v_new[:, e - n:e].contiguous()) for i, ((_, n), e) in enumerate(zip(batch, ends))]
    else:
        st["out"] = torch.empty(q.shape, dtype=torch.float32, device="cuda")
        st["roots"] = [h[files[f][1]] for f, _ in batch] if kind == "beam" else None
        if layers == 1 and kind != "beam":
            st["batch"] = ctx.prepare_batch(st["kv"], st["n"], q[0], k_new[0], v_new[0], st["out"][0])
        else:
            st["args"] = [(q[i], k_new[i], v_new[i], st["out"][i]) for i in range(layers)]
    torch.cuda.synchronize()                     # the rows appended above are freed on return
    return st


def run(st):
    ctx, stream, kind = st["ctx"], st["sess"].stream, st["kind"]
    if kind == "prune":
        for h in ctx.kv_extract_batch(st["kv"], None, stream, st["idx"], st["off"]):
            ctx.kv_remove(h)
        return {"pool": st["pool"]}
    if kind == "append":
        for h, n, k, v in st["parts"]:
            ctx.kv_append(h, n, k, v, stream)
        ctx.kv_truncate(st["kv"], st["lens"])
        return {"pool": st["pool"]}
    if kind == "beam":
        kv = [ctx.kv_fork(r) for r in st["roots"]]
        ctx.pred_batch(kv, st["n"], *st["args"][0], stream)
        for h in kv:
            ctx.kv_remove(h)
    else:
        if st["layers"] == 1:
            ctx.pred_prepared(st["batch"], stream)
        else:
            ctx.pred_begin(st["kv"], st["n"], stream)
            for i, a in enumerate(st["args"]):
                ctx.pred_layer(i, *a, stream)
        ctx.kv_truncate(st["kv"], st["lens"])
    return {"out": st["out"], "pool": st["pool"]}


def exact(case, seed):
    if case["kind"] in ("prune", "append"):
        return None                              # rows are moved bit for bit; nothing is computed
    files, batch, own, K, V, q, k_new, v_new = _inputs(case, seed)
    s = _shape(case)
    G, at = s.n_q_heads // s.n_kv_heads, np.concatenate([[0], np.cumsum(own)]).tolist()
    out = torch.empty(q.shape, dtype=torch.float64, device="cuda")
    for i in range(q.shape[0]):
        t = 0
        for f, n in batch:
            root = files[f][1]
            rows = lambda X, new: torch.cat(([X[i, at[root]:at[root + 1]]] if root is not None else []) + [X[i, at[f]:at[f + 1]], new[i, t:t + n]]).double().permute(1, 0, 2).contiguous()  # noqa: E731
            k, v = rows(K, k_new), rows(V, v_new)                                                  # [Hkv, L + n, D]
            x = q[i, t:t + n].double().view(n, s.n_kv_heads, G, s.head_dim).permute(1, 0, 2, 3).reshape(s.n_kv_heads, n * G, s.head_dim)
            S = torch.matmul(x, k.transpose(1, 2).contiguous()) / s.head_dim ** 0.5
            if n > 1:
                seen = torch.arange(k.shape[1], device="cuda")[None, :] <= k.shape[1] - n + torch.arange(n, device="cuda")[:, None]
                S.masked_fill_(~seen.repeat_interleave(G, 0)[None], float("-inf"))
            o = torch.matmul(torch.softmax(S, -1), v)
            out[i, t:t + n] = o.view(s.n_kv_heads, n, G, s.head_dim).permute(1, 0, 2, 3).reshape(n, s.n_q_heads, s.head_dim)
            t += n
    return {"out": out, "pool": None}


def work(case):
    files, batch = _layout(case)
    s, layers = _shape(case), case.get("layers", 1)
    token = s.kv_bytes_per_token
    if case["kind"] == "append":
        return {"bytes": 2 * token * sum(n for _, n in batch), "flops": 0}
    if case["kind"] == "prune":                  # about half of the tokens after the first page: read and written
        return {"bytes": 2 * token * sum(max(0, n - P) / 2 for n, _ in files), "flops": 0}
    stored = sum(n - (files[root][0] if root is not None else 0) for n, root in files)      # shared pages once
    T, es = sum(n for _, n in batch), 4 if s.dtype == "f32" else 2
    pairs = sum(n * files[f][0] + n * (n + 1) // 2 for f, n in batch)
    row = s.n_q_heads * s.head_dim
    return {"bytes": layers * (stored * token + T * (2 * token + row * (es + 4))), "flops": layers * 4 * row * pairs}


def tolerance(case):
    """Stored rows ("pool", whole numbers) are the same bits.  Outputs: about four times what the path shows against
    64 bits where softmax weights are rounded to 16 bits for the matrix cores (2.3e-4); 32-bit sums in fp32 storage."""
    if case["kind"] in ("prune", "append"):
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 1e-4, "differ": 0.0}
    return {"rel": 1e-3, "max": 1e-2, "differ": 0.0}
