"""The work that a user of the CFGzip library has it do, as measurable cases.

Five kinds, each through the public entry points of ``paper_2605_29986_amd``:

  decode   one decode step: class masks expanded and applied to the logits, sampled tokens mapped to
           their representatives (``cfgzip_decode_step``)
  engine   one decode step of the byte-automaton engine: states advanced on the sampled tokens, logits
           masked with the states' class masks (``cfgzip_engine_step``)
  classes  the pre-computation for a deterministic byte automaton: signatures, then classes
  grammar  the pre-computation for a grammar in Greibach normal form: displacement sets, then classes
  nfa      the pre-computation for a non-deterministic byte automaton: relations, then classes

Inputs are seeded and synthetic.  Vocabularies, automata and grammars come from ``synthetic_inputs``;
their sizes are those of the repository's configurations and tests, or lie between them.  A program keeps
its workspaces from call to call, so ``prepare`` makes them; results that the binding allocates when it
is not handed a tensor are allocated by it here too.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_2605_29986_amd as cfgzip
from synthetic_inputs.dfa import make_json_like_dfa, make_lexer_dfa
from synthetic_inputs.grammar import make_clike_gnf, make_json_gnf
from synthetic_inputs.nfa import add_transitions, nfa_from_dfa
from synthetic_inputs.vocab import make_vocab_mixture, make_vocab_uniform

NINF = float("-inf")


def _words(n):
    return (n + 31) // 32


def listed():
    return [
        # interactive use: one sequence, a small vocabulary; what counts is the latency of one launch
        {"name": "decode_b1", "kind": "decode", "B": 1, "V": 32_000, "C": 683, "dtype": "bf16",
         "stride": 32_000, "bits": False},
        # a small batch whose sampler wants fp32 logits
        {"name": "decode_b16_f32", "kind": "decode", "B": 16, "V": 128_256, "C": 1_460, "dtype": "f32",
         "stride": 128_256, "bits": False},
        # an odd vocabulary with contiguous rows: no row but the first starts on a 16-byte boundary
        {"name": "decode_b64_odd", "kind": "decode", "B": 64, "V": 50_003, "C": 3_001, "dtype": "bf16",
         "stride": 50_003, "bits": True},
        # the serving batch of the benchmark's decode workload, with the token mask as by-product
        {"name": "decode_b256", "kind": "decode", "B": 256, "V": 128_256, "C": 8_000, "dtype": "bf16",
         "stride": 128_256, "bits": True},
        # the closed decode loop of the byte-automaton engine at a medium batch
        {"name": "engine_b64", "kind": "engine", "B": 64, "V": 128_256, "S": 1_024, "cap": 32,
         "dtype": "bf16", "bits": False},
        # the smallest class build: a tiny vocabulary and automaton, all launches and the final wait
        {"name": "classes_4k", "kind": "classes", "V": 4_096, "S": 24, "cap": 8, "rows": True},
        # a medium vocabulary against a lexer whose table fits in LDS, signature rows stored
        {"name": "classes_32k", "kind": "classes", "V": 32_000, "S": 256, "cap": 16, "rows": True},
        # a large vocabulary against a lexer that does not fit in LDS, signature rows stored
        {"name": "classes_128k", "kind": "classes", "V": 128_256, "S": 1_024, "cap": 32, "rows": True},
        # the largest vocabulary and automaton, signatures hashed on the fly
        {"name": "classes_152k", "kind": "classes", "V": 151_936, "S": 4_096, "cap": 64, "rows": False},
        # a JSON grammar over a large vocabulary, rows long enough for every set
        {"name": "grammar_json_128k", "kind": "grammar", "grammar": "json", "V": 128_256, "cap": 32,
         "row_len": 1_024},
        # a statement grammar over a medium vocabulary with the shortest rows
        {"name": "grammar_clike_32k", "kind": "grammar", "grammar": "clike", "V": 32_000, "cap": 16,
         "row_len": 256},
        # a lexer with overlapping rules before it is made deterministic
        {"name": "nfa_32k", "kind": "nfa", "V": 32_000, "S": 256, "cap": 16},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("decode", "decode", "decode", "engine", "classes", "classes", "classes", "grammar",
                       "grammar", "nfa"))
    if kind == "decode":
        dtype = rng.choice(("bf16", "f32"))
        V = _log_int(rng, 4_096, 160_000)
        most = 256 * 128_256 // V if dtype == "bf16" else 128 * 128_256 // V
        B = _log_int(rng, 1, min(256, most))
        C = _log_int(rng, 24, min(V // 4, 16_000))
        # rows as the LM head leaves them: contiguous, or padded to whole multiples of 64 columns
        stride = V if rng.random() < 0.5 else (V + 63) // 64 * 64
        return {"kind": "decode", "B": B, "V": V, "C": C, "dtype": dtype, "stride": stride,
                "bits": rng.random() < 0.5}
    if kind == "engine":
        V = _log_int(rng, 4_096, 130_000)
        return {"kind": "engine", "B": _log_int(rng, 1, 256), "V": V, "S": _log_int(rng, 128, 1_024),
                "cap": rng.choice((16, 32)), "dtype": rng.choice(("bf16", "f32")) if V < 60_000 else "bf16",
                "bits": rng.random() < 0.5}
    if kind == "classes":
        V = _log_int(rng, 2_000, 152_000)
        if V < 6_000 and rng.random() < 0.5:
            return {"kind": "classes", "V": V, "S": 24, "cap": 8, "rows": rng.random() < 0.5}
        S = _log_int(rng, 128, 4_096)
        rows = rng.random() < 0.5 and 2 * V * S <= 262_000_000
        return {"kind": "classes", "V": V, "S": S, "cap": rng.choice((16, 32, 64)), "rows": rows}
    if kind == "grammar":
        return {"kind": "grammar", "grammar": rng.choice(("json", "clike")), "V": _log_int(rng, 2_000, 128_000),
                "cap": rng.choice((16, 32)), "row_len": rng.choice((256, 512, 1_024))}
    S = _log_int(rng, 128, 1_024)
    most = 262_000_000 // (4 * S * _words(S))
    return {"kind": "nfa", "V": _log_int(rng, 1_000, max(1_000, min(32_000, most))), "S": S,
            "cap": rng.choice((16, 32))}


# ---------------------------------------------------------------- inputs


def _class_map(rng, V, C):
    """A class map with the heavy-tailed class sizes of real builds: ids by first appearance,
    the representative one member of the class."""
    weights = 1.0 / np.arange(1, C + 1) ** 1.1
    cls = np.concatenate([np.arange(C), rng.choice(C, size=V - C, p=weights / weights.sum())])
    rng.shuffle(cls)
    _, first, inv = np.unique(cls, return_index=True, return_inverse=True)
    rank = np.empty(C, np.int64)
    rank[np.argsort(first, kind="stable")] = np.arange(C)
    rep = np.empty(C, np.int32)
    rep[rank] = first
    return rank[inv].astype(np.int32), rep


def _logits(B, stride, dtype, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn((B, stride), device="cuda", generator=gen) * 2.0
    return x.to(torch.bfloat16) if dtype == "bf16" else x


def _token_mask_buffer(case):
    if not case["bits"]:
        return None
    return torch.empty((case["B"], _words(case["V"])), dtype=torch.int32, device="cuda")


def _automaton(case, seed):
    """(table uint16 [S][256], keywords)"""
    if case["S"] == 24:
        return make_json_like_dfa(seed), []
    return make_lexer_dfa(seed, case["S"])


def _vocabulary(case, seed, keywords):
    if case.get("S") == 24:
        v = make_vocab_uniform(seed, V=case["V"], max_len=case["cap"])
    else:
        v = make_vocab_mixture(seed, case["V"], case["cap"], 0.1 if case["cap"] > 16 else 0.0, keywords)
    return torch.from_numpy(v.tok_bytes).cuda(), torch.from_numpy(v.tok_off).cuda()


def _representatives(V):
    """The buffer a program hands over for the representatives: as many entries as there may be classes;
    those behind the last class keep what they hold."""
    return torch.full((V,), -1, dtype=torch.int32, device="cuda")


def _bytes(n):
    return torch.empty(n, dtype=torch.uint8, device="cuda")


def _prepare_decode(case, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    B, V, C = case["B"], case["V"], case["C"]
    c, r = _class_map(rng, V, C)
    return {
        "logits": _logits(B, case["stride"], case["dtype"], seed),
        "cls_bits": torch.from_numpy(rng.integers(-2**31, 2**31, size=(B, _words(C)), dtype=np.int64)
                                     .astype(np.int32)).cuda(),
        "tok": torch.from_numpy(rng.integers(0, V, size=B).astype(np.int32)).cuda(),
        "c": torch.from_numpy(c).cuda(), "r": torch.from_numpy(r).cuda(),
        "tok_bits": _token_mask_buffer(case),
    }


def _prepare_engine(case, seed):
    """The tables of a grammar given as a byte automaton, made the way a program makes them, and the
    state of a running batch: live states, and for each an allowed token that was sampled from it."""
    rng = np.random.Generator(np.random.PCG64(seed))
    B, V, S = case["B"], case["V"], case["S"]
    table, keywords = _automaton(case, seed + 500)
    tb, to = _vocabulary(case, seed, keywords)
    tt = torch.from_numpy(table).cuda()
    ws = _bytes(cfgzip.load_library().cfgzip_signatures_workspace_bytes(V, S))
    _, h = cfgzip.cfgzip_signatures(tb, to, tt, want_sig=False, workspace=ws)
    c, r, C, _ = cfgzip.cfgzip_build_classes(tb, to, tt, None, h, signatures_workspace=ws)
    rb, ro = cfgzip.cfgzip_representative_vocabulary(tb, to, r)
    sig_rep, _ = cfgzip.cfgzip_signatures(rb, ro, tt, want_hash=False)
    live = rng.random(S) < 0.3
    live[0] = False
    while True:
        more = live | live[table].any(axis=1)
        if (more == live).all():
            break
        live = more
    state_mask = cfgzip.cfgzip_state_masks(sig_rep, torch.from_numpy(live.astype(np.uint8)).cuda())
    ok = live[sig_rep.cpu().numpy()]  # [C][S]: class allowed in state
    c_host = c.cpu().numpy()
    states = rng.choice(np.nonzero(live & ok.any(axis=0))[0], size=B)
    tok = np.empty(B, np.int32)
    for b in range(B):
        tok[b] = rng.choice(np.nonzero(ok[c_host, states[b]])[0])
    return {
        "logits": _logits(B, V, case["dtype"], seed), "state_mask": state_mask, "C": C, "c": c,
        "sig_rep": sig_rep, "tok": torch.from_numpy(tok).cuda(),
        "states": torch.from_numpy(states.astype(np.int32)).cuda(), "tok_bits": _token_mask_buffer(case),
    }


def _prepare_classes(case, seed):
    lib = cfgzip.load_library()
    V, S = case["V"], case["S"]
    table, keywords = _automaton(case, seed + 500)
    tb, to = _vocabulary(case, seed, keywords)
    return {
        "tb": tb, "to": to, "table": torch.from_numpy(table).cuda(), "rows": case["rows"],
        "r": _representatives(V), "ws_sig": _bytes(lib.cfgzip_signatures_workspace_bytes(V, S)),
        "ws_build": _bytes(lib.cfgzip_build_classes_workspace_bytes(V, S)),
    }


def _prepare_grammar(case, seed):
    lib = cfgzip.load_library()
    g = make_json_gnf() if case["grammar"] == "json" else make_clike_gnf()
    # words of a program in the vocabulary, as the grammars' own keywords are
    tb, to = _vocabulary(case, seed, [b"true", b"false", b"null", b"if", b"while", b"return"])
    return {
        "tb": tb, "to": to, "grammar": [torch.from_numpy(x).cuda() for x in g.arrays()], "N": g.N,
        "row_len": case["row_len"], "r": _representatives(case["V"]),
        "ws": _bytes(lib.cfgzip_displacements_workspace_bytes(case["V"], g.N, g.P)),
        "ws_build": _bytes(lib.cfgzip_build_classes_workspace_bytes(case["V"], case["row_len"])),
    }


def _prepare_nfa(case, seed):
    lib = cfgzip.load_library()
    S, W = case["S"], _words(case["S"])
    table, keywords = make_lexer_dfa(seed + 500, S)
    nfa = add_transitions(nfa_from_dfa(table), seed + 501, 0.10)
    tb, to = _vocabulary(case, seed, keywords)
    return {
        "tb": tb, "to": to, "nfa": torch.from_numpy(nfa.view(np.int32)).cuda(), "r": _representatives(case["V"]),
        "ws_build": _bytes(lib.cfgzip_build_classes_workspace_bytes(case["V"], 2 * S * W)),
    }


def prepare(case, seed):
    make = {"decode": _prepare_decode, "engine": _prepare_engine, "classes": _prepare_classes,
            "grammar": _prepare_grammar, "nfa": _prepare_nfa}
    s = make[case["kind"]](case, seed)
    s["case"] = case
    return s


# ---------------------------------------------------------------- one pass


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "decode":
        rep = cfgzip.cfgzip_decode_step(s["logits"], s["cls_bits"], s["c"], case["C"], s["tok"], s["r"],
                                        tok_bits_out=s["tok_bits"], V=case["V"])
        return {"logits": s["logits"], "tok_bits": s["tok_bits"], "rep": rep}
    if kind == "engine":
        states = cfgzip.cfgzip_engine_step(s["logits"], s["state_mask"], s["C"], s["c"], s["sig_rep"],
                                           s["tok"], s["states"], tok_bits_out=s["tok_bits"])
        return {"logits": s["logits"], "tok_bits": s["tok_bits"], "states": states}
    if kind == "classes":
        sig, h = cfgzip.cfgzip_signatures(s["tb"], s["to"], s["table"], want_sig=s["rows"],
                                          workspace=s["ws_sig"])
        c, _, C, _ = cfgzip.cfgzip_build_classes(s["tb"], s["to"], s["table"], sig, h, rep_of_class=s["r"],
                                                 workspace=s["ws_build"], signatures_workspace=s["ws_sig"])
        return {"sig": None if sig is None else sig.view(torch.int16), "hash": h, "c": c, "r": s["r"], "C": C}
    if kind == "grammar":
        rows, h, status = cfgzip.cfgzip_displacements(s["tb"], s["to"], *s["grammar"], s["N"],
                                                      row_len=s["row_len"], workspace=s["ws"])
        c, _, C, _ = cfgzip.cfgzip_build_classes(s["tb"], s["to"], None, rows, h, rep_of_class=s["r"],
                                                 workspace=s["ws_build"])
        return {"rows": rows.view(torch.int16), "hash": h, "status": status, "c": c, "r": s["r"], "C": C}
    rel, h = cfgzip.cfgzip_nfa_signatures(s["tb"], s["to"], s["nfa"])
    V, S, W = rel.shape
    c, _, C, _ = cfgzip.cfgzip_build_classes(s["tb"], s["to"], None, rel.view(torch.uint16).reshape(V, 2 * S * W),
                                             h, rep_of_class=s["r"], workspace=s["ws_build"])
    return {"rel": rel, "hash": h, "c": c, "r": s["r"], "C": C}


# ---------------------------------------------------------------- what a pass cannot do without


def _vocabulary_bytes(V, cap):
    if cap == 8:
        mean = 4.5  # lengths uniform on 1..8
    else:
        mean = (1.0 - 0.8 ** cap) / 0.2  # lengths min(Geom(0.2), cap)
    return V * mean + 8 * (V + 1)


def work(case):
    """Bytes: every input read once, every output written once.  There is no arithmetic to speak of:
    table look-ups, comparisons and selects."""
    kind, V = case["kind"], case["V"]
    if kind in ("decode", "engine"):
        B = case["B"]
        C = case["C"] if kind == "decode" else 1_000  # class masks are a small share either way
        n = 2 * B * V * (2 if case["dtype"] == "bf16" else 4) + 4 * V + 4 * B * _words(C) + 16 * B
        if case["bits"]:
            n += 4 * B * _words(V)
        return {"bytes": n, "flops": 0}
    n = _vocabulary_bytes(V, case["cap"]) + 8 * V + 4 * V  # hashes and class ids out
    if kind == "classes":
        n += 512 * case["S"] + (2 * V * case["S"] if case["rows"] else 0)
    elif kind == "grammar":
        n += 2 * V * case["row_len"] + 4 * V
    else:
        n += 4 * (V + 256) * case["S"] * _words(case["S"])
    return {"bytes": n, "flops": 0}


def tolerance(case):
    # logits are copied or set to -inf, everything else is whole numbers
    return "exact"


def exact(case, seed):
    """Masked logits by plain torch; the other outputs are whole numbers and compared as they are."""
    if case["kind"] != "decode":
        return None
    s = _prepare_decode(case, seed)
    V = case["V"]
    bit = s["c"].long()
    allowed = (s["cls_bits"].long()[:, bit // 32] >> (bit % 32)) & 1
    z = s["logits"].double()
    z[:, :V] = torch.where(allowed.bool(), z[:, :V], torch.full_like(z[:, :V], NINF))
    return {"logits": z, "tok_bits": None, "rep": None}
