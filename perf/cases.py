"""What is measured of this library: bursts of decode steps as a serving loop runs them.

A pass puts the batch's parse stacks back to where they stood after a warm-up text and then runs STEPS
decode steps through the public calls, each step on logits of its own (a model writes new ones for every
step).  The texts, and with them stacks, masks and tokens, come from decoding random logits under the
grammar on the device, so every sequence is somewhere else in a document of its own.

A case names
  call      which calls make a step:
              step    advance_fill_apply_mask: advance by the sampled token, next mask, masked logits
              greedy  advance_fill_argmax: the same with the greedy choice, fed back as the next token
              topk    advance_fill_mask, then apply_mask_topk: a sampler that takes the k best
              split   fill_mask, apply_mask, advance: a server that samples between its own calls
              jump    jump_forward, fill_apply_mask, advance: forced text is emitted without the model
  grammar   arithmetic | json | schema (fixed keys, one grammar) | mixed (eight schemas in one batch)
            | right_recursive (JSON with right-recursive lists, cycle-aware stacks)
  vocab, batch
  stride    elements between two rows of logits: the vocabulary itself (what a projection to an odd
            vocabulary gives) or more (a padded projection)
  graph     the burst is captured once as a HIP graph and replayed, as servers do with small batches
  k         length of the top-k list
"""
import functools

import numpy as np
import torch

from paper_2506_03887_amd import Pre3, apply_mask

STEPS = 8          # decode steps of a pass
WARM = 24          # tokens of each sequence before the pass
CAP = 256          # stack entries per sequence
MAX_JUMP = 32      # forced bytes a call may emit

ARITHMETIC = r'''
E ::= E "+" T | T
T ::= T "*" F | F
F ::= "(" E ")" | "a"
'''

_VALUE = r'''
json     ::= ws value
value    ::= object ws | array ws | string ws | number ws | "true" ws | "false" ws | "null" ws
object   ::= "{" ws "}" | "{" ws members "}"
member   ::= string ws ":" ws value
array    ::= "[" ws "]" | "[" ws elements "]"
'''

# %s: the lists of the lexical part, left- or right-recursive
_LEXICAL = r'''
string   ::= "\"" chars "\""
char     ::= plain | "\\" escape
plain    ::= [^"\\\x00-\x1f]
escape   ::= simple | "u" hex hex hex hex
simple   ::= ["\\/bfnrt]
hex      ::= [0-9a-fA-F]
number   ::= sign int frac exp
sign     ::= "" | "-"
int      ::= "0" | onenine | onenine digits
digit    ::= [0-9]
onenine  ::= [1-9]
frac     ::= "" | "." digits
exp      ::= "" | e esign digits
e        ::= [eE]
esign    ::= "" | [+\-]
wsc      ::= [ \t\n\r]
'''
_LEFT = r'''
chars    ::= "" | chars char
digits   ::= digit | digits digit
ws       ::= "" | ws wsc
'''
_RIGHT = r'''
chars    ::= "" | char chars
digits   ::= digit | digit digits
ws       ::= "" | wsc ws
'''
JSON = _VALUE + r'''
members  ::= member | members "," ws member
elements ::= value | elements "," ws value
''' + _LEXICAL + _LEFT
RIGHT_RECURSIVE = _VALUE + r'''
members  ::= member | member "," ws members
elements ::= value | value "," ws elements
''' + _LEXICAL + _RIGHT


def _words(rng, n):
    """n lowercase words with different first letters, so that one byte tells them apart."""
    first = rng.permutation(26)[:n]
    return ["".join(chr(97 + int(c)) for c in (f, *rng.integers(0, 26, size=int(rng.integers(2, 9))))) for f in first]


def _schema(seed, keys, depth):
    """An object with fixed keys in fixed order; values cycle through integer, number, one of eight words,
    truth value, string, nested object and list of objects (`depth` levels)."""
    rng = np.random.default_rng(seed)
    rules, names = [], iter(range(10_000))

    def obj(level, n):
        name, members = "o%d" % next(names), []
        for i, key in enumerate(_words(rng, n)):
            kind = ("intv", "number", "enum", "boolv", "string", "obj", "arr")[i % (7 if level < depth else 5)]
            if kind == "enum":
                kind = "e%d" % next(names)
                rules.append("%s ::= %s" % (kind, " | ".join('"\\"%s\\""' % w for w in _words(rng, 8))))
            elif kind == "obj":
                kind = obj(level + 1, max(3, n // 2))
            elif kind == "arr":
                inner, at = obj(level + 1, max(2, n // 3)), next(names)
                kind = "a%d" % at
                rules.append('%s ::= "[" ws "]" | "[" ws i%d "]"' % (kind, at))
                rules.append('i%d ::= %s ws | i%d "," ws %s ws' % (at, inner, at, inner))
            at = next(names)
            rules.append('k%d ::= "\\"%s\\"" ws ":" ws %s ws' % (at, key, kind))
            members.append("k%d" % at)
        rules.append('%s ::= "{" ws %s "}"' % (name, ' "," ws '.join(members)))
        return name

    top = obj(1, keys)
    return "\n".join(["root ::= ws %s ws" % top, *rules]) + '\nintv ::= sign int\nboolv ::= "true" | "false"\n' + _LEXICAL + _LEFT


def _grammars(name):
    if name == "mixed":
        return [_schema(50 + i, *shape) for i, shape in
                enumerate(((5, 1), (8, 2), (12, 2), (14, 3), (16, 3), (16, 3), (18, 3), (19, 3)))]
    return [{"arithmetic": ARITHMETIC, "json": JSON, "right_recursive": RIGHT_RECURSIVE}.get(name) or _schema(40, 12, 3)]


@functools.lru_cache(maxsize=None)
def _vocabulary(grammar, n):
    """(bytes, offsets) of n tokens, the last one the end of sequence.  JSON-like text: the 256 single bytes,
    then byte strings of geometric length (mean 4, at most 32) from a text-like distribution."""
    rng = np.random.default_rng(n)
    if grammar == "arithmetic":
        lens = np.concatenate([np.ones(8, dtype=np.int64), rng.integers(1, 5, size=n - 9), [0]])
        alphabet = np.frombuffer(b"a+*()b- ", dtype=np.uint8)
        text = alphabet[np.concatenate([np.arange(8), rng.integers(0, 8, size=int(lens.sum()) - 8)])]
    else:
        p = np.zeros(256)
        for group, share in ((b"abcdefghijklmnopqrstuvwxyz", .32), (b"ABCDEFGHIJKLMNOPQRSTUVWXYZ", .08), (b"0123456789", .15),
                             (b'"{}[]:,', .25), (b" ", .08), (b"\n", .02), (b"-._/\\+eEtn", .10)):
            p[list(group)] += share / len(group)
        lens = np.concatenate([np.ones(256, dtype=np.int64), np.minimum(rng.geometric(0.25, size=n - 257), 32), [0]])
        text = np.concatenate([np.arange(256, dtype=np.uint8), rng.choice(256, size=int(lens.sum()) - 256, p=p / p.sum()).astype(np.uint8)])
    return np.append(text, np.uint8(0)), np.concatenate([[0], np.cumsum(lens)])


def _case(name, call, grammar, vocab, batch, stride=None, graph=False, k=0):
    case = dict(call=call, grammar=grammar, vocab=vocab, batch=batch, stride=stride or vocab, graph=graph, k=k)
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest batch and vocabulary, one call after the other: all launches and latency; rows of odd length
        _case("step arithmetic 4", "step", "arithmetic", 513, 4),
        # one user's document: the latency of a decode step with a large vocabulary
        _case("step json 1 graph", "step", "json", 128256, 1, graph=True),
        # a small server with a small vocabulary
        _case("step json 64 graph", "step", "json", 32000, 64, graph=True),
        # the common serving batch: one sequence per compute unit
        _case("step json 256", "step", "json", 128256, 256),
        # structured output of a fixed schema (sparse masks), a large batch and vocabulary
        _case("step schema 512", "step", "schema", 152064, 512),
        # the largest: throughput serving
        _case("step json 2048", "step", "json", 128256, 2048),
        # greedy decoding, at the common batch and on one somewhat larger than the chip with cycle-aware stacks
        _case("greedy json 256", "greedy", "json", 128256, 256),
        _case("greedy right 320", "greedy", "right_recursive", 128256, 320),
        # sampling from the k best: a full and a small batch
        _case("topk json 256", "topk", "json", 128256, 256, k=50),
        _case("topk schema 16 graph", "topk", "schema", 152064, 16, graph=True, k=50),
        # a vocabulary of odd size without padding: every row starts at another alignment
        _case("split json 96 ragged", "split", "json", 100003, 96),
        # many schemas in one batch, forced text emitted without the model
        _case("jump mixed 128", "jump", "mixed", 128256, 128),
    ]


def _spread(rng, lo, hi):
    """An integer of lo..hi, spread over its logarithm."""
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    call = rng.choice(("step", "step", "greedy", "topk", "split", "jump"))
    grammar = rng.choice(("arithmetic", "json", "json", "schema", "mixed", "right_recursive"))
    vocab = _spread(rng, 16, 4096) if grammar == "arithmetic" else _spread(rng, 600, 200_000)
    batch = _spread(rng, 1, min(2048, 2048 * 128256 // (2 if call in ("step", "greedy") else 4) // vocab))
    stride = rng.choice((vocab, vocab, -(-vocab // 64) * 64, -(-vocab // 8) * 8))
    return _case(None, call, grammar, vocab, batch, stride, graph=batch <= 64 and rng.random() < 0.5,
                 k=rng.randint(1, 64) if call == "topk" else 0)


def prepare(case, seed):
    dev = torch.device("cuda")
    V, B, call = case["vocab"], case["batch"], case["call"]
    text, offsets = _vocabulary(case["grammar"], V)
    lib = Pre3(_grammars(case["grammar"]), text, offsets, V - 1, stack_cap=CAP, compact_cycles=case["grammar"] == "right_recursive")
    gen = torch.Generator(device=dev).manual_seed(seed)
    # stacks, states, lengths and error codes of the batch lie in one buffer, so that one copy restores them
    live = torch.zeros(B * (CAP + 3), dtype=torch.int32, device=dev)
    data, rest = live[: B * CAP].view(B, CAP), live[B * CAP:].view(3, B)
    states, length, err = rest[0], rest[1], rest[2]
    which = torch.randint(lib.n_grammars, (B,), generator=gen, device=dev)
    states.copy_(torch.tensor([lib.initial_state(g) for g in range(lib.n_grammars)], dtype=torch.int32, device=dev)[which])
    data[:, 0] = states
    length.fill_(1)
    lib.bind_state(states, data, length, err)
    mask = torch.zeros((B, lib.words), dtype=torch.int32, device=dev)
    tokens = torch.zeros((STEPS + 1, B), dtype=torch.int32, device=dev)
    logits = torch.empty((STEPS, B, case["stride"]), dtype=torch.bfloat16, device=dev)[:, :, :V]
    jumped = torch.zeros((STEPS, B, MAX_JUMP), dtype=torch.uint8, device=dev), torch.zeros((STEPS, B), dtype=torch.int32, device=dev)
    top = torch.zeros((STEPS, B, max(1, case["k"])), dtype=torch.int32, device=dev), \
        torch.zeros((STEPS, B, max(1, case["k"])), dtype=torch.bfloat16, device=dev)
    ends = call in ("step", "greedy", "topk")       # these calls restart a sequence that ends its text
    start = None
    for s in range(WARM + STEPS):                   # decode random logits: every allowed token equally likely
        x = logits[s % STEPS]
        x.normal_(generator=gen)
        # a text that may end does so half of the time (in the pass itself only where the call restarts it)
        x[:, V - 1] = torch.randint(2, (B,), generator=gen, device=dev).to(x.dtype) * 60 - 30 if ends or s < WARM else -30
        if s == WARM:
            start = live.clone()
        if call == "jump":
            lib.jump_forward(jumped[0][0], jumped[1][0])
        lib.fill_mask(states, data, length, mask)
        tok = tokens[max(0, s - WARM)]
        lib.apply_mask_argmax(x, mask, tok)
        if ends or s < WARM:
            lib.advance_fill_mask(tok, mask, restart_on_eos=True)
        else:
            lib.advance(tok)
    state = dict(call=call, lib=lib, live=live, start=start, states=states, data=data, length=length, err=err, mask=mask,
                 tokens=tokens, logits=logits, jumped=jumped, top=top, vocab=V, graph=None)
    if case["graph"]:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _burst(state)
        torch.cuda.current_stream().wait_stream(side)
        for x in logits:                            # what the burst has masked
            x.normal_(generator=gen)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            _burst(state)
        state["graph"] = graph
    return state


def _burst(s):
    lib, call, mask, tokens = s["lib"], s["call"], s["mask"], s["tokens"]
    states, data, length = s["states"], s["data"], s["length"]
    torch.add(s["start"], 0, out=s["live"])
    for i in range(STEPS):
        x = s["logits"][i]
        if call == "step":
            lib.advance_fill_apply_mask(tokens[i], mask, x, restart_on_eos=True)
        elif call == "greedy":
            lib.advance_fill_argmax(tokens[i], mask, x, tokens[i + 1], restart_on_eos=True)
        elif call == "topk":
            lib.advance_fill_mask(tokens[i], mask, restart_on_eos=True)
            lib.apply_mask_topk(x, mask, s["top"][0][i], s["top"][1][i])
        elif call == "split":
            lib.fill_mask(states, data, length, mask)
            apply_mask(x, mask, s["vocab"])
            lib.advance(tokens[i])
        else:
            lib.jump_forward(s["jumped"][0][i], s["jumped"][1][i])
            lib.fill_apply_mask(states, data, length, mask, x)
            lib.advance(tokens[i])


def run(state):
    if state["graph"] is not None:
        state["graph"].replay()
    else:
        _burst(state)
    out = {n: state[n] for n in ("states", "data", "length", "err", "mask")}
    if state["call"] == "greedy":
        out["tokens"] = state["tokens"]
    elif state["call"] == "topk":
        out["top"] = state["top"]
    else:
        out["logits"] = state["logits"]
        if state["call"] == "jump":
            out["jumped"] = state["jumped"]
    return out


def work(case):
    """Per step: the logits read (and, where they are masked in place, written), the mask row written.  The stacks
    and the tables are small beside that.  Selecting and moving bits only: no arithmetic to speak of."""
    pairs = STEPS * case["batch"] * case["vocab"]
    return {"bytes": pairs * ((2 if case["call"] in ("greedy", "topk") else 4) + 1 / 8), "flops": pairs}


def tolerance(case):
    return "exact"    # whole numbers, bits, and logits that are kept or replaced, never computed
