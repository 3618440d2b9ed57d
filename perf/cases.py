"""Timing cases of the token-mask path: what a serving engine has this library do, from the smallest call to the largest.

A case is a dict of plain values; `prepare` makes what the engine has in hand before the call, `run` is one pass through
the public entry points.  The paths:

  decode   one decoding step with the matchers on the device: accept the sampled tokens, fill the next-token bitmask,
           apply it to the logits
  host     the same step with the matchers on the host (fill uploads their parser contexts)
  compile  a request with a grammar of its own: compile it, re-admit its sequences (replay the tokens they have already),
           fill their masks
  pool     several requests with overlapping tool sets compiled into one cross-grammar pool, then one mask for each
  jit      a request compiled just in time: a few decoding steps, the fills building what they reach

Grammars: `nested` one JSON schema with objects, arrays and enums; `tools` free text with tagged calls of a tool set;
`records` a list of up to 1,000 records with bounded strings and integers.  Vocabularies and documents are synthetic; the
vocabulary stands for the tokenizer, which a program loads once, and does not depend on the seed.
"""
import functools
import math
import random

import numpy as np
import torch

import gen
import paper_2601_04426_amd as xg
from gen.grammars import sub_object_type, tool_schema

PERIOD = 64          # decoding steps after which a state's token table starts over
RESET = -2           # in the token table: the slot starts a new sequence


def listed():
    return [
        # one interactive sequence: nothing but launches and latency
        dict(name="decode_single", path="decode", grammar="nested", size=20, grammars=1, vocab=32000, batch=1, dtype="f32"),
        # a small chat batch, free text with tool calls
        dict(name="decode_chat_tools", path="decode", grammar="tools", size=16, grammars=1, vocab=128256, batch=16, dtype="bf16"),
        # structured extraction with a middle-sized vocabulary
        dict(name="decode_nested", path="decode", grammar="nested", size=20, grammars=1, vocab=32000, batch=64, dtype="f32"),
        # a vocabulary size that no vector width divides, a batch that is no power of two
        dict(name="decode_odd_vocab", path="decode", grammar="nested", size=12, grammars=1, vocab=50021, batch=37, dtype="bf16"),
        # a full batch in which every request brings a tool set of its own
        dict(name="decode_mixed_tools", path="decode", grammar="tools", size=12, grammars=16, vocab=151936, batch=256, dtype="f32"),
        # the largest batch, long bounded lists
        dict(name="decode_records", path="decode", grammar="records", size=1000, grammars=1, vocab=151936, batch=1024, dtype="bf16"),
        # parsers on the host: a small batch in a loop that must not allocate, and a large one
        dict(name="host_small", path="host", grammar="nested", size=20, grammars=1, vocab=128256, batch=8, dtype="bf16", noalloc=True),
        dict(name="host_records", path="host", grammar="records", size=1000, grammars=1, vocab=151936, batch=256, dtype="bf16", noalloc=False),
        # a request's grammar compiled from scratch: one schema, and one tool set
        dict(name="compile_nested", path="compile", grammar="nested", size=20, grammars=1, vocab=32000, batch=4),
        dict(name="compile_tools", path="compile", grammar="tools", size=16, grammars=1, vocab=128256, batch=8),
        # requests that draw their tools from one library, compiled one after another into a shared pool
        dict(name="pool_requests", path="pool", grammar="tools", size=12, grammars=8, vocab=151936, batch=8),
        # just-in-time compilation of a long bounded list and the first steps of a batch
        dict(name="jit_records", path="jit", grammar="records", size=1000, grammars=1, vocab=151936, batch=64, steps=12, prebuild=5),
    ]


def _between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(("decode", "decode", "decode", "host", "compile", "compile", "pool", "jit"))
    grammar = "tools" if path == "pool" else rng.choice(("nested", "tools", "records"))
    vocab = _between(rng, 2000, 152000) | 1 if rng.random() < 0.4 else 32 * _between(rng, 64, 4748)
    size = {"nested": rng.randint(6, 30), "tools": rng.randint(4, 24), "records": _between(rng, 50, 1000)}[grammar]
    case = dict(path=path, grammar=grammar, size=size, grammars=1, vocab=vocab)
    if path == "decode":
        if grammar == "tools" and rng.random() < 0.5:
            case.update(grammars=rng.randint(2, 12), size=rng.randint(4, 12))
        case.update(batch=max(case["grammars"], _between(rng, 1, 1024)), dtype=rng.choice(("bf16", "f32")))
        if case["dtype"] == "f32":
            case["batch"] = min(case["batch"], 512)
    elif path == "host":
        case.update(batch=_between(rng, 1, 256), dtype=rng.choice(("bf16", "f32")))
        case.update(noalloc=case["batch"] * ((vocab + 31) // 32) <= 1 << 19 and rng.random() < 0.4)
    elif path == "compile":
        case.update(batch=rng.randint(1, 8))
    elif path == "pool":
        case.update(grammars=rng.randint(2, 8), size=rng.randint(4, 12))
        case["batch"] = case["grammars"]
    else:
        case.update(batch=_between(rng, 4, 64), steps=rng.randint(4, 12), prebuild=rng.choice((0, 5, 10)))
    return case


@functools.lru_cache(maxsize=2)
def _vocabulary(size):
    """(synthetic tokenizer, segmenter, library handle): loaded once by a program, whatever its requests."""
    v = gen.make_vocab(size, size ^ 0x5EED, "bpe")
    return v, gen.Segmenter(v), xg.Vocab(v.tokens, v.eos_id, v.special_ids)


def _name(rng):
    return "".join(rng.choice("abcdefghijklmnopqrstuvwxyz_") for _ in range(rng.randint(4, 12)))


def _names(rng, n):
    out = []
    while len(out) < n:
        x = _name(rng)
        if x not in out:
            out.append(x)
    return out


def _free_text(rng):
    return "".join(chr(rng.choice((10, *range(0x20, 0x3C), *range(0x3D, 0x7F)))) for _ in range(rng.randint(0, 30)))


def _nested(rng, n_props):
    schema = gen.nested_schema(rng, n_props, 3)
    return gen.schema_to_ebnf(schema), lambda r: gen.render_value(gen.random_value(schema, r), r)


def _tools(rng, tools):
    """tools: (name, argument schema, rule name).  Free text of any bytes in which "<function=NAME>" starts a call."""
    pairs = ", ".join('("<function=%s>", %s)' % (name, rule) for name, _, rule in tools)
    lines, seen = ["root ::= TagDispatch(%s)" % pairs], set()
    for name, schema, rule in tools:
        lines.append('%s ::= %s "</function>"' % (rule, schema.rule))
        for line in gen.schema_to_ebnf(schema, root_rule="unused", with_basic=False).splitlines()[1:]:
            if line.split(" ::= ", 1)[0] not in seen:
                seen.add(line.split(" ::= ", 1)[0])
                lines.append(line)

    def text(r):
        out = _free_text(r)
        for _ in range(r.randint(1, 3)):
            name, schema, _ = r.choice(tools)
            out += "<function=%s>%s</function>%s" % (name, gen.render_value(gen.random_value(schema, r), r), _free_text(r))
        return out
    return "\n".join(lines) + "\n" + gen.grammars.BASIC_RULES, text


def _tool_library(rng, n, shared=0):
    subs = [sub_object_type(rng, i) for i in range(shared)] or None
    return [(name, tool_schema(rng, "t%d_" % i, subs), "tool%d" % i) for i, name in enumerate(_names(rng, n))]


def _records(rng, most):
    fields = [(n, rng.choice(("str", "int"))) for n in _names(rng, rng.randint(2, 4))]
    item = ' ws "," ws '.join('"\\"%s\\"" ws ":" ws %s' % f for f in fields)
    ebnf = ('root ::= "[" ws item (ws "," ws item){0,%d} ws "]"\n'
            'item ::= "{" ws %s ws "}"\n'
            'str ::= "\\"" [^"\\\\\\x00-\\x1F]{0,64} "\\""\n'
            'int ::= "-"? [0-9]{1,19}\n'
            'ws ::= [ \\n\\t]*\n' % (most - 1, item))

    def value(r, kind):
        if kind == "str":
            return '"%s"' % "".join(chr(r.choice((0xE9, *range(0x23, 0x5C), *range(0x5D, 0x7F)))) for _ in range(r.randint(0, 64)))
        return r.choice(("", "", "-")) + "".join(r.choice("0123456789") for _ in range(r.randint(1, 19)))

    def text(r):
        ws = lambda: r.choice(("", "", "", " ", "\n"))  # noqa: E731
        body = ["{" + ws() + (ws() + "," + ws()).join('"%s":%s%s' % (n, ws(), value(r, k)) for n, k in fields) + "}" for _ in range(r.randint(1, 8))]
        return "[" + ws() + (ws() + "," + ws()).join(body) + ws() + "]"
    return ebnf, text


def _requests(case, rng):
    """The case's grammars, as (EBNF text, sampler of documents)."""
    if case["grammar"] == "nested":
        return [_nested(rng, case["size"]) for _ in range(case["grammars"])]
    if case["grammar"] == "records":
        return [_records(rng, case["size"]) for _ in range(case["grammars"])]
    n = case["grammars"]
    library = _tool_library(rng, case["size"] if n == 1 else 3 * case["size"], shared=0 if n == 1 else 16)
    return [_tools(rng, library if n == 1 else rng.sample(library, case["size"])) for _ in range(n)]


def _streams(rng, seg, text, eos, n, length):
    """`n` token streams: a reset, a document, the end of sequence, a reset, the next document, ..., cut at `length`."""
    out = []
    for _ in range(n):
        s = []
        while len(s) < length:
            s += [RESET] + seg.segment(text(rng).encode("utf-8"), rng) + [eos]
        out.append(s[:length])
    return out


def _decode_tables(case, rng, seg, samplers, eos):
    """(tokens that bring every slot to its starting depth, one row a step; the table of the steps that follow): slot b
    goes round a stream of PERIOD tokens from a random place on."""
    G, B = case["grammars"], case["batch"]
    streams = [_streams(rng, seg, text, eos, min(24, -(-B // G)), PERIOD) for text in samplers]
    mine = [rng.choice(streams[b % G]) for b in range(B)]
    at = [rng.randrange(PERIOD) for _ in range(B)]
    lead = np.full((max(at), B), -1, dtype=np.int32)
    table = np.empty((PERIOD, B), dtype=np.int32)
    for b in range(B):
        lead[:at[b], b] = mine[b][:at[b]]
        table[:, b] = mine[b][at[b]:] + mine[b][:at[b]]
    return lead, table


def _compile_all(vocab, requests, stream):
    pool = xg.Pool() if len(requests) > 1 else None
    return [xg.compile_grammar(vocab, ebnf, pool=pool, stream=stream) for ebnf, _ in requests]


def prepare(case, seed):
    rng = random.Random(seed)
    tok, seg, vocab = _vocabulary(case["vocab"])
    dev = torch.device("cuda")
    stream = torch.cuda.current_stream().cuda_stream
    V, W, B, G = vocab.size, vocab.words, case["batch"], case["grammars"]
    requests = _requests(case, rng)
    s = dict(path=case["path"], vocab=vocab, V=V, W=W, B=B, stream=stream,
             bitmask=torch.zeros((case.get("steps", 1), B, W) if case["path"] == "jit" else (B, W), dtype=torch.int32, device=dev))
    if case["path"] in ("decode", "host"):
        dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        g = torch.Generator(device=dev).manual_seed(seed)
        s.update(logits=torch.randn((B, V), generator=g, dtype=dtype, device=dev), dtype=xg.XG2_BF16 if case["dtype"] == "bf16" else xg.XG2_F32, step=0)
        caches = _compile_all(vocab, requests, stream)
        lead, table = _decode_tables(case, rng, seg, [text for _, text in requests], tok.eos_id)
        if case["path"] == "decode":
            db = xg.DeviceBatch(vocab, B)
            for k, c in enumerate(caches):
                db.assign(c, rows=list(range(k, B, G)), stream=stream)
            s.update(batch=db, status=torch.zeros(B, dtype=torch.int32, device=dev), ids=list(torch.from_numpy(table).to(dev).unbind(0)))
            for row in torch.from_numpy(lead).to(dev).unbind(0):
                db.accept_tokens(row.data_ptr(), s["status"].data_ptr(), stream)
        else:
            matchers = [xg.Matcher(caches[b % G]) for b in range(B)]
            s.update(matchers=matchers, batch=xg.MatcherBatch(matchers), noalloc=case["noalloc"])
            s["resets"] = [np.nonzero(row == RESET)[0].tolist() for row in table]
            s["ids"] = list(np.where(table == RESET, -1, table))
            for row in lead:
                _host_accept(s, np.nonzero(row == RESET)[0].tolist(), np.where(row == RESET, -1, row))
    elif case["path"] == "jit":
        s.update(ebnf=requests[0][0], steps=case["steps"], prebuild=case["prebuild"])
        docs = [seg.segment(requests[0][1](rng).encode("utf-8"), rng) + [tok.eos_id] for _ in range(min(24, B))]
        mine = [rng.choice(docs) for _ in range(B)]
        at = [rng.randrange(min(len(d), 24)) for d in mine]
        s["replay"] = [d[:a] for d, a in zip(mine, at)]
        # a document that ends within the steps: its sequence is done and gets no further token
        s["ids"] = [np.array([d[a + k] if a + k < len(d) else -1 for d, a in zip(mine, at)], dtype=np.int32) for k in range(case["steps"])]
    else:
        s["ebnf"] = [ebnf for ebnf, _ in requests]
        s["replay"] = []
        for b in range(B):
            ids = seg.segment(requests[b % G][1](rng).encode("utf-8"), rng)
            s["replay"].append(ids[:rng.randrange(min(len(ids), 24))])
    return s


def _host_accept(s, resets, ids):
    for b in resets:
        s["matchers"][b].reset()
    return s["batch"].accept_tokens(ids)


def run(s):
    return {"decode": _run_decode, "host": _run_host, "compile": _run_compile, "pool": _run_pool, "jit": _run_jit}[s["path"]](s)


def _run_decode(s):
    k = s["step"]
    s["step"] = (k + 1) % PERIOD
    s["batch"].accept_tokens(s["ids"][k].data_ptr(), s["status"].data_ptr(), s["stream"])
    s["batch"].fill_next_token_bitmask(s["bitmask"].data_ptr(), s["W"], s["stream"])
    xg.apply_token_bitmask(s["logits"].data_ptr(), s["dtype"], s["B"], s["V"], s["V"], s["bitmask"].data_ptr(), s["W"], s["stream"])
    return {"status": s["status"], "bitmask": s["bitmask"], "logits": s["logits"]}


def _run_host(s):
    k = s["step"]
    s["step"] = (k + 1) % PERIOD
    status = _host_accept(s, s["resets"][k], s["ids"][k])
    fill = xg.fill_next_token_bitmask_noalloc if s["noalloc"] else xg.fill_next_token_bitmask
    fill(s["batch"], s["bitmask"].data_ptr(), s["W"], s["stream"])
    xg.apply_token_bitmask(s["logits"].data_ptr(), s["dtype"], s["B"], s["V"], s["V"], s["bitmask"].data_ptr(), s["W"], s["stream"])
    return {"status": status, "bitmask": s["bitmask"], "logits": s["logits"]}


def _readmit(s, caches):
    """The requests' sequences with the tokens they have already; row b belongs to cache b modulo their number."""
    matchers = [xg.Matcher(caches[b % len(caches)]) for b in range(s["B"])]
    for m, ids in zip(matchers, s["replay"]):
        for t in ids:
            m.accept_token(t)
    return matchers


def _first_masks(s, caches):
    matchers = _readmit(s, caches)
    xg.fill_next_token_bitmask(matchers, s["bitmask"].data_ptr(), s["W"], s["stream"])
    # what the engine logs of each build: planes, and the bits of all of them
    stats = [c.stats for c in caches]
    return {"bitmask": s["bitmask"], "built": [int(t.built) for t in stats], "accepted": [int(t.n_accepted) for t in stats],
            "uncertain": [int(t.n_uncertain) for t in stats]}


def _run_compile(s):
    return _first_masks(s, [xg.compile_grammar(s["vocab"], s["ebnf"][0], stream=s["stream"])])


def _run_pool(s):
    pool = xg.Pool()
    return _first_masks(s, [xg.compile_grammar(s["vocab"], ebnf, pool=pool, stream=s["stream"]) for ebnf in s["ebnf"]])


def _run_jit(s):
    cache = xg.compile_grammar(s["vocab"], s["ebnf"], stream=s["stream"], jit=True, jit_prebuild=s["prebuild"])
    batch = xg.MatcherBatch(_readmit(s, [cache]))
    for k in range(s["steps"]):
        xg.fill_next_token_bitmask(batch, s["bitmask"][k].data_ptr(), s["W"], s["stream"])
        status = batch.accept_tokens(s["ids"][k])
    return {"bitmask": s["bitmask"], "status": status, "planes": cache.num_planes()}


def work(case):
    """Bytes: a decoding step writes the mask, reads it and writes the logits once (masked ones are overwritten, mixed
    vectors are read too: counted as one pass over the logits for JSON, where nearly everything is masked, and as a
    quarter of one for free text, where nearly everything is allowed).  A compile reads the token bytes and writes two bits
    per (plane, token); planes per grammar as counted on these generators: about 28 a property of a nested schema, 330 a
    tool on its own and 200 a tool in a shared pool, 150 for a list of records (a just-in-time build reaches about 40)."""
    V, B = case["vocab"], case["batch"]
    W = (V + 31) // 32
    if case["path"] in ("decode", "host"):
        logits = B * V * (2 if case["dtype"] == "bf16" else 4) * (0.25 if case["grammar"] == "tools" else 1.0)
        return {"bytes": 2 * B * W * 4 + logits, "flops": 0}
    if case["path"] == "jit":
        planes = 40
    else:
        planes = case["grammars"] * {"nested": 28 * case["size"], "tools": (330 if case["path"] == "compile" else 200) * case["size"], "records": 150}[case["grammar"]]
    return {"bytes": case["grammars"] * 6 * V + planes * 2 * W * 4 + case.get("steps", 1) * B * W * 4, "flops": 0}


def tolerance(case):
    """Masks, states and counts are whole numbers, and masked logits are either left alone or minus infinity."""
    return "exact"
