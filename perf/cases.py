"""The work that a user of this framework has it do: the listed cases and the ranges they stand for.

A case is one call of the operator (Alg. 1), or of one of its stages, through `binding`:

  op "full"    selection and block-sparse attention (`ba_att`), or, with `buffers`, the two calls on
               workspaces and outputs that the program keeps, as a serving loop does
  op "select"  the selection stage alone (`basa_select`): its lists are reused over several steps
  op "dense"   the dense baseline (`basa_dense_attn`)
  op "decode"  a block of new queries against the keys and values of everything before it
               (`ba_att` with L_q < L_k)
  op "varlen"  sequences of different lengths, packed token-major (`ba_att_varlen`)

Values come from the seeded generators of `synth` (diffusion-LM, multimodal and video shaped).
"""
import math

import torch

from paper_2605_19726_amd import binding as bd
from paper_2605_19726_amd import synth

DEVICE = "cuda"
DEFAULTS = dict(op="full", kind="lowrank", dtype="bf16", heads_q=32, heads_kv=32, L=16384, L_q=0, n_seq=0, d=128,
                block=128, sparsity=0.5, mass_target=0.0, beta=1.0, sort=bd.SORT_QK, causal=False, segments=False,
                buffers=False, token_major=False, image_side=0, frames=0, frame_h=0, frame_w=0)


def _case(**kw):
    c = dict(DEFAULTS)
    c.update(kw)
    return c


def listed():
    return [
        # the fp32 parity workload: one head, the smallest call anyone makes; launches and host work count
        _case(name="tiny_f32", kind="salient", dtype="f32", heads_q=1, heads_kv=1, L=1024, d=64, block=64),
        # a short prompt of a small model, ragged last block, head dimension 64: still latency
        _case(name="short_d64", heads_q=8, heads_kv=8, L=2472, d=64, block=64),
        # an fp32 layer of ordinary size (evaluation in full precision)
        _case(name="layer_f32_4k", dtype="f32", heads_q=8, heads_kv=8, L=4096),
        # the shortest of the length sweep at its highest sparsity: stages of comparable size
        _case(name="dlm_16k_s90", L=16384, sparsity=0.9),
        # a block of new tokens of a diffusion LM with grouped heads against a long context
        _case(name="decode_256_of_32k", op="decode", heads_q=32, heads_kv=8, L=32768, L_q=256, sparsity=0.75),
        # six prompts of different lengths in one packed batch
        _case(name="varlen_6", op="varlen", heads_q=16, heads_kv=16, L=24576, n_seq=6),
        # the dense baseline at the shortest length of the sweep
        _case(name="dense_16k", op="dense", L=16384),
        # the autoregressive variant
        _case(name="causal_32k", L=32768, causal=True),
        # selection alone on the 32K workload (blocks of 64): computed once, reused by later steps
        _case(name="select_32k_b64", op="select", L=32768, block=64),
        # multimodal LM: grouped heads, image and text sorted apart, blocks kept by cumulative mass
        _case(name="multimodal_64k", kind="multimodal", heads_q=32, heads_kv=8, L=65536, image_side=128, segments=True,
              sparsity=0.25, mass_target=0.5),
        # video diffusion transformer: ragged length, token-major output for the projection that follows
        _case(name="video_75k_s75", kind="video", heads_q=40, heads_kv=40, L=75600, frames=21, frame_h=60, frame_w=60,
              sparsity=0.75, buffers=True, token_major=True),
        # the headline workload
        _case(name="dlm_128k", L=131072, buffers=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes log-uniform (most of them no multiple of anything), the options of its family."""
    family = rng.choice(["f32", "f32_layer", "short", "dlm", "dlm", "decode", "varlen", "dense", "causal", "select",
                         "multimodal", "video"])
    d, block = rng.choice([64, 128]), rng.choice([64, 128])
    s = rng.choice([0.5, 0.75, 0.9])
    c = _case(d=d, block=block, sparsity=s)
    if family == "f32":
        h = rng.randint(1, 2)
        c.update(kind="salient", dtype="f32", heads_q=h, heads_kv=h, L=_log(rng, 300, 2048))
    elif family == "f32_layer":
        h = rng.randint(2, 8)
        c.update(dtype="f32", heads_q=h, heads_kv=h, L=_log(rng, 1024, 6000))
    elif family == "short":
        kv = rng.choice([2, 4, 8])
        c.update(heads_q=kv * rng.choice([1, 4]), heads_kv=kv, L=_log(rng, 500, 8192))
    elif family == "dlm":
        h = rng.choice([16, 24, 32])
        c.update(heads_q=h, heads_kv=h, L=_log(rng, 8192, 100000), buffers=rng.random() < 0.5,
                 token_major=rng.random() < 0.5)
    elif family == "decode":
        c.update(op="decode", heads_q=32, heads_kv=rng.choice([8, 32]), L=_log(rng, 4096, 100000), L_q=_log(rng, 32, 1024))
    elif family == "varlen":
        h = rng.choice([8, 16, 32])
        c.update(op="varlen", heads_q=h, heads_kv=h // rng.choice([1, 4]), L=_log(rng, 6000, 48000), n_seq=rng.randint(2, 10))
    elif family == "dense":
        h = rng.choice([8, 16, 32])
        c.update(op="dense", heads_q=h, heads_kv=h // rng.choice([1, 4]), L=_log(rng, 1024, 40000))
    elif family == "causal":
        h = rng.choice([8, 16, 32])
        c.update(heads_q=h, heads_kv=h, L=_log(rng, 2048, 60000), causal=True, sort=rng.choice([bd.SORT_NONE, bd.SORT_QK]))
    elif family == "select":
        c.update(op="select", heads_q=32, heads_kv=rng.choice([8, 32]), L=_log(rng, 8192, 131072),
                 beta=rng.choice([0.0, 1.0]))
    elif family == "multimodal":
        side = rng.randint(32, 128)
        c.update(kind="multimodal", heads_q=32, heads_kv=8, image_side=side, L=side * side + _log(rng, 2000, 49152),
                 segments=True, sparsity=0.25, mass_target=rng.choice([0.5, 0.7]))
    else:
        h = rng.choice([12, 24, 40])
        t, hh, ww = rng.randint(5, 21), rng.randint(24, 60), rng.randint(24, 60)
        c.update(kind="video", heads_q=h, heads_kv=h, d=128, block=128, frames=t, frame_h=hh, frame_w=ww, L=t * hh * ww,
                 buffers=True, token_major=True)
    return c


def _lengths(c):
    """Sequence lengths of a packed batch: unequal shares of L tokens, none a multiple of the block."""
    n, L = c["n_seq"], c["L"]
    weight = [1.0 + 2.5 * ((7 * i) % n) for i in range(n)]
    lens = [max(1, int(L * x / sum(weight))) for x in weight]
    lens[0] += L - sum(lens)
    return lens


def _workload(c, seed, L):
    return synth.Workload(str(c.get("name", "drawn")), int(seed), c["kind"], c["heads_q"], c["heads_kv"], L, c["d"], c["block"],
                          c["dtype"], (c["sparsity"],), salient_frac=0.02 if c["kind"] == "lowrank" else 0.0,
                          salient_count=3 if c["kind"] == "salient" else 0, image_side=c["image_side"],
                          video_thw=(c["frames"], c["frame_h"], c["frame_w"]))


def prepare(case, seed):
    c = dict(case)
    w = _workload(c, seed, c["L"])
    q, k, v = synth.make_qkv(w, device=DEVICE)
    if c["op"] == "decode":
        q = q[:, :, -c["L_q"]:].contiguous()              # the newest tokens
    st = dict(c=c, q=q, k=k, v=v, segments=synth.segments_of(w) if c["segments"] else None)
    if c["op"] == "varlen":
        st["cu"] = [0]
        for n in _lengths(c):
            st["cu"].append(st["cu"][-1] + n)
        for t in ("q", "k", "v"):                         # token-major: [tokens, heads, d]
            st[t] = st[t][0].permute(1, 0, 2).contiguous()
    out = torch.empty(q.shape[0], q.shape[2], q.shape[1], q.shape[3], dtype=q.dtype, device=q.device).permute(0, 2, 1, 3) \
        if c["token_major"] else None
    if c["buffers"]:
        p = bd.params(c["block"], c["sparsity"], c["beta"], c["sort"], mass_target=c["mass_target"], causal=c["causal"])
        st["ws_sel"] = torch.empty(bd.select_workspace_size(q, k, p), dtype=torch.uint8, device=q.device)
        st["ws_att"] = torch.empty(bd.attn_workspace_size(q, k, p), dtype=torch.uint8, device=q.device)
        st["sel"] = bd.basa_select(q, k, c["block"], c["sparsity"], c["beta"], c["sort"], ws=st["ws_sel"],
                                   mass_target=c["mass_target"], causal=c["causal"])
        out = torch.empty_like(q) if out is None else out
    st["out"] = out
    return st


def _lists(c, sel):
    """What a selection writes: the columns of a row past its count are left as they were, so they are
    returned only where every row keeps the full count."""
    r = dict(row_count=sel.row_count, perm_q=sel.perm_q, perm_k=sel.perm_k)
    if c["mass_target"] == 0.0 and not c["causal"]:
        r["row_cols"] = sel.row_cols
    for n in ("mask_bits", "row_mass"):
        if getattr(sel, n) is not None:
            r[n] = getattr(sel, n)
    return r


def run(st):
    c, q, k, v = st["c"], st["q"], st["k"], st["v"]
    B, s = c["block"], c["sparsity"]
    if c["op"] == "dense":
        return bd.basa_dense_attn(q, k, v, B)
    if c["op"] == "varlen":
        return bd.ba_att_varlen(q, k, v, st["cu"], B, s)
    if c["op"] == "select":
        return _lists(c, bd.basa_select(q, k, B, s, c["beta"], c["sort"]))
    if c["buffers"]:
        sel = bd.basa_select(q, k, B, s, c["beta"], c["sort"], ws=st["ws_sel"], out=st["sel"], mass_target=c["mass_target"],
                             causal=c["causal"])
        out = bd.basa_sparse_attn(q, k, v, sel.row_count, sel.row_cols, B, sel.perm_q, sel.perm_k, ws=st["ws_att"],
                                  out=st["out"], causal=c["causal"])
    else:
        out, sel = bd.ba_att(q, k, v, B, s, c["beta"], c["sort"], mass_target=c["mass_target"], segments=st["segments"],
                             out=st["out"], causal=c["causal"])
    return dict(out=out, **_lists(c, sel))


def work(case):
    """Every input read once, every output written once; 4 d flops per token pair of the kept blocks and the
    3d-long products of the block map."""
    c = case
    e = 4 if c["dtype"] == "f32" else 2
    B, d, hq, hk = c["block"], c["d"], c["heads_q"], c["heads_kv"]
    seqs = [(n, n) for n in _lengths(c)] if c["op"] == "varlen" else [(c["L_q"] or c["L"], c["L"])]
    nbytes = flops = 0.0
    for lq, lk in seqs:
        nq, nk = -(-lq // B), -(-lk // B)
        kappa = max(1, nk - int(c["sparsity"] * nk + 1e-9))
        select, attend = c["op"] != "dense", c["op"] != "select"
        keep = 1.0 if c["op"] == "dense" else kappa / nk
        if c["mass_target"] > 0.0:
            keep = min(keep, c["mass_target"])            # the fewest blocks that carry the mass: at most this share
        if c["causal"]:
            keep *= 0.5
        nbytes += (hq * lq + hk * lk) * d * e
        if attend:
            nbytes += (hk * lk + hq * lq) * d * e
            flops += 4.0 * hq * lq * lk * keep * d
        if select:
            nbytes += hq * nq * (kappa + 1) * 4 + (hq * lq + hk * lk) * 4
            flops += 2.0 * hq * nq * nk * (3 * d if c["beta"] else d)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Permutations are exact; a block whose score ties with its row's threshold to within the rounding of
    the fp32 logits may be another one, which moves a few list entries and the output rows of that block."""
    if case["op"] == "select":
        return {"rel": 1e-5, "max": 1e-3, "differ": 1e-3}
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3, "differ": 1e-3}
    return {"rel": 1e-2, "max": 0.5, "differ": 1e-3}
