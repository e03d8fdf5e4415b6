"""GPU stage checks through the production kernels, against the oracle.

tfhe_debug_mod_switch_batch runs the pre-combination and modulus-switch
kernel on its own; tfhe_debug_cmux_batch runs the blind-rotation kernel for
one CMux step from a caller-given accumulator and key row, in the launch
shape a bootstrap batch of the same size takes.  That lets a test drive the
external product's worst case -- every gadget digit at -Bg/2 against key
parts at their largest magnitude -- through the kernels that the bootstraps
use, bit for bit against the oracle's schoolbook CMux.
"""
import sys

import numpy as np
import pytest

import oracle
from paper_1911_07101_amd import tfhe, workloads as wl

pytestmark = pytest.mark.gpu

M32 = 1 << 32


def say(msg):
    print(f"[gpu-stages] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    return _t


_KEYS = {}


def keys_for(cfg_name):
    if cfg_name not in _KEYS:
        cfg = wl.CONFIGS[cfg_name]
        say(f"keygen {cfg_name}")
        sk, ek = tfhe.tfhe_keygen_from_seed(cfg["params"], cfg["key_seed"], 0)
        _KEYS[cfg_name] = (sk, ek, oracle.Keys(cfg["params"], cfg["key_seed"]))
    return _KEYS[cfg_name]


def u32(a):
    return (np.asarray(a, dtype=np.int64) % M32).astype(np.uint32)


# ------------------------------------------------------------ modulus switch

@pytest.mark.parametrize("cfg_name", ["toy", "tfhe128_nand", "lut3_n2048"])
def test_mod_switch_stage_every_word(torch, cfg_name):
    """Every word of a batch in the timed launch shape, with planted ties
    (rounded up), words one below a tie and words that wrap to 0, against
    the oracle's modulus switch word by word."""
    p = wl.CONFIGS[cfg_name]["params"]
    n, N = p["n"], p["N"]
    sk, ek, ok = keys_for(cfg_name)
    B = {"toy": 37, "tfhe128_nand": 4096 + 3, "lut3_n2048": 8192 + 5}[cfg_name]
    rng = np.random.default_rng(91)
    x = rng.integers(0, M32, (B, n + 1), dtype=np.uint64).astype(np.uint32)
    step = M32 // (2 * N)
    k = rng.integers(0, 2 * N, (B, n + 1))
    kind = rng.integers(0, 4, (B, n + 1))
    x = np.where(kind == 0, u32(k * step + step // 2),                     # a tie: rounds up to k + 1
                 np.where(kind == 1, u32(k * step + step // 2 - 1),        # just below: k
                          np.where(kind == 2, u32(M32 - step // 2), x)))    # wraps to 0
    say(f"mod switch stage {cfg_name} B={B}")
    got = tfhe.tfhe_debug_mod_switch_batch(ek, tfhe.to_device(x)).cpu().numpy().view(np.uint16)
    ref = oracle.mod_switch_array(x, N)
    assert got.shape == (B, n + 1) and np.array_equal(got.astype(np.uint32), ref)
    assert (ref[kind == 2] == 0).all() and (ref[kind == 0] == (k[kind == 0] + 1) % (2 * N)).all()


@pytest.mark.parametrize("gate", ["NAND", "XOR", "ANDNY"])
def test_mod_switch_stage_after_gate_combination(torch, gate):
    """The gate's pre-combination followed by the modulus switch, at the
    128-bit parameters, rows sampled across the batch, against the oracle's
    combination and modulus switch."""
    p = wl.CONFIGS["tfhe128_nand"]["params"]
    sk, ek, ok = keys_for("tfhe128_nand")
    B = 4096 + 3
    rng = np.random.default_rng(92)
    a, b = rng.integers(0, 2, B), rng.integers(0, 2, B)
    ca = tfhe.tfhe_encrypt_torus(sk, 93, tfhe.encode_bits(a), 0)
    cb = tfhe.tfhe_encrypt_torus(sk, 93, tfhe.encode_bits(b), B)
    say(f"gate {gate} + mod switch B={B}")
    got = tfhe.tfhe_debug_mod_switch_batch(ek, tfhe.to_device(ca), gate, tfhe.to_device(cb)).cpu().numpy()
    got = got.view(np.uint16).astype(np.uint32)
    for r in np.linspace(0, B - 1, 24).astype(int):
        comb = oracle.gate_combine(ok.p, gate, ca[r], cb[r])
        assert np.array_equal(got[r], oracle.mod_switch_array(comb, p["N"])), r


# ----------------------------------------------------------------- one CMux

def digit_word(p, digit):
    """A coefficient D whose signed gadget decomposition is `digit` in all l
    positions (the rounding bits below the last digit are 0)."""
    l, bg = p["l"], p["bg_bit"]
    half = 1 << (bg - 1)
    rnd = 1 << (31 - l * bg) if l * bg < 32 else 0
    # the decomposition adds Bg/2 in every position and the rounding bit, so
    # the digit field is digit + Bg/2
    return u32(sum((digit + half) << (32 - j * bg) for j in range(1, l + 1)) - sum(
        half << (32 - j * bg) for j in range(1, l + 1)) - rnd)


def acc_for_difference(D):
    """An accumulator ACC with X^N ACC - ACC = -2 ACC = D (D even)."""
    D = np.asarray(D, dtype=np.int64)
    assert (D % 2 == 0).all()
    return u32(-(D // 2))


# key rows: every coefficient one value, chosen by its signed 16-bit parts
# (low, high) as the library splits it: (-2^15, -2^15 + 1), (2^15 - 1, 2^15 - 1)
# and (-2^15, 2^15), the largest magnitudes the split produces
KEY_WORDS = {"parts_neg": 0x80008000, "parts_pos": 0x7FFF7FFF, "parts_mixed": 0x7FFF8000}


def key_row(p, pattern, ok):
    N, l = p["N"], p["l"]
    if pattern == "eval_key_row":
        return np.ascontiguousarray(ok.bk_view()[0]).ravel()
    if pattern == "alternating":
        w = np.where(np.arange(N) % 2 == 0, KEY_WORDS["parts_neg"], KEY_WORDS["parts_pos"]).astype(np.uint32)
        return np.tile(w, 2 * l * 2)
    return np.full(2 * l * 2 * N, KEY_WORDS[pattern], np.uint32)


KEY_ROW_PATTERNS = ("parts_neg", "parts_pos", "parts_mixed", "alternating", "eval_key_row")


@pytest.mark.parametrize("cfg_name,B", [("tfhe128_nand", 4096), ("tfhe128_nand", 1000), ("tfhe128_nand", 250),
                                        ("lut3_n2048", 1027), ("lut3_n2048", 600), ("lut3_n2048", 250), ("toy", 37)])
@pytest.mark.parametrize("pattern", KEY_ROW_PATTERNS)
def test_one_cmux_worst_case(torch, cfg_name, B, pattern):
    """One CMux in every launch shape at 256 CUs (N = 1024: 4096 accumulators
    in 8-wave blocks, 1000 in one-wave blocks, 250 a block each; N = 2048:
    1027 in blocks of four ciphertexts with a last round of teams, 600 in
    one-ciphertext blocks, 250 in teams; N = 256: 37 a block each), bit for
    bit against the oracle's CMux.  The
    first accumulators rotate by N with every coefficient of both
    polynomials chosen so that every gadget digit is -Bg/2 (the largest
    magnitude), then every digit Bg/2 - 1, then digits alternating between
    the two by coefficient, then a descending ramp; the rest are random with
    random rotations.  Against key rows whose parts are all at the largest
    magnitude with one sign, of opposite signs, alternating, or the eval
    key's own first row, this is the 2l-term sum of the transform's error
    bound at or near its worst case."""
    p = wl.CONFIGS[cfg_name]["params"]
    N, l, bg = p["N"], p["l"], p["bg_bit"]
    sk, ek, ok = keys_for(cfg_name)
    rng = np.random.default_rng(list(KEY_ROW_PATTERNS).index(pattern) + N)
    half = 1 << (bg - 1)
    d_min, d_max = digit_word(p, -half), digit_word(p, half - 1)
    # the planted differences decompose as intended
    assert oracle.decompose(l, bg, int(d_min)) == [-half] * l
    assert oracle.decompose(l, bg, int(d_max)) == [half - 1] * l
    acc = rng.integers(0, M32, (B, 2, N), dtype=np.uint64).astype(np.uint32)
    abar = rng.integers(0, 2 * N, B).astype(np.uint32)
    alt = np.where(np.arange(N) % 2 == 0, d_min, d_max)
    ramp = u32(np.linspace(-(1 << 31), (1 << 31) - 2, N).astype(np.int64) & ~1)
    planted = {0: np.full(N, d_min), 1: np.full(N, d_max), 2: alt, 3: ramp,
               B - 1: np.full(N, d_min)}
    for r, D in planted.items():
        acc[r] = acc_for_difference(np.broadcast_to(D, (2, N)))
        abar[r] = N
    row = key_row(p, pattern, ok)
    say(f"one CMux {cfg_name} key {pattern} B={B}")
    got = tfhe.to_host(tfhe.tfhe_debug_cmux_batch(ek, row, tfhe.to_device(abar), tfhe.to_device(acc)))
    check = sorted(set(planted) | set(np.linspace(4, B - 2, 10).astype(int)))
    for r in check:
        ref = oracle.cmux_row(p, row, int(abar[r]), acc[r])
        assert np.array_equal(got[r], ref), f"accumulator {r}"


def test_one_cmux_matches_blind_rotation_step(torch):
    """The stage check with the eval key's own rows reproduces the blind
    rotation: starting from (0, X^{-bbar} v) and applying the CMux of rows
    0..3 in turn gives the oracle's accumulator after four steps (toy)."""
    p = wl.CONFIGS["toy"]["params"]
    N = p["N"]
    sk, ek, ok = keys_for("toy")
    rng = np.random.default_rng(94)
    B = 9
    acc = np.zeros((B, 2, N), np.uint32)
    acc[:, 1] = oracle.gate_testvec(N)
    ref = acc.copy()
    for i in range(4):
        abar = rng.integers(0, 2 * N, B).astype(np.uint32)
        row = np.ascontiguousarray(ok.bk_view()[i]).ravel()
        acc = tfhe.to_host(tfhe.tfhe_debug_cmux_batch(ek, row, tfhe.to_device(abar), tfhe.to_device(acc)))
        ref = np.stack([oracle.cmux(ok, i, int(abar[c]), ref[c]) for c in range(B)])
        assert np.array_equal(acc, ref), i


def test_stage_checks_reject_bad_arguments(torch):
    sk, ek, ok = keys_for("toy")
    p = wl.CONFIGS["toy"]["params"]
    N = p["N"]
    acc = tfhe.to_device(np.zeros((2, 2, N), np.uint32))
    abar = tfhe.to_device(np.zeros(2, np.uint32))
    with pytest.raises(ValueError):  # a key row of the wrong size
        tfhe.tfhe_debug_cmux_batch(ek, np.zeros(5, np.uint32), abar, acc)
    with pytest.raises(tfhe.TfheError) as ei:  # output on top of the input
        tfhe.tfhe_debug_cmux_batch(ek, np.zeros(2 * p["l"] * 2 * N, np.uint32), abar, acc, out=acc)
    assert ei.value.rc == tfhe.TFHE_EINVAL and "overlaps" in str(ei.value)
    with pytest.raises(tfhe.TfheError) as ei:
        tfhe.tfhe_debug_mod_switch_batch(ek, tfhe.to_device(np.zeros((2, p["n"] + 1), np.uint32)), gate=17,
                                         cb=tfhe.to_device(np.zeros((2, p["n"] + 1), np.uint32)))
    assert ei.value.rc == tfhe.TFHE_EINVAL


# --------------------------------------------------------- buffer placement

def test_overlapping_buffers_are_rejected(torch):
    """Inputs, outputs and workspace of one call must not overlap: a ReLU
    computed in place (whose windows would read sign words that earlier
    windows overwrote), an iReLU writing over its error bits, a gate writing
    over an operand, and a workspace inside the output are refused before
    any launch."""
    p = wl.CONFIGS["toy"]["params"]
    sk, ek, ok = keys_for("toy")
    row = p["n"] + 1
    x = tfhe.to_device(np.zeros((3, 8, row), np.uint32))
    cases = {
        "relu in place": lambda: tfhe.glyph_relu_batch(ek, x, 8, y=x),
        "irelu over delta": lambda: tfhe.glyph_irelu_batch(ek, x, x, out=x),
        "gate over an operand": lambda: tfhe.tfhe_gate_bootstrap_batch(ek, "AND", x[0], x[1], out=x[1]),
        "workspace in the output": lambda: tfhe.tfhe_gate_bootstrap_batch(
            ek, "AND", x[0], x[1], out=x[2], workspace=x[2].view(torch.uint8)),
    }
    for name, call in cases.items():
        with pytest.raises(tfhe.TfheError) as ei:
            call()
        assert ei.value.rc == tfhe.TFHE_EINVAL and "overlaps" in str(ei.value), name
    # a partial overlap of two rows in one buffer
    ext = tfhe.to_device(np.zeros((3, p["N"] + 1), np.uint32))
    with pytest.raises(tfhe.TfheError) as ei:
        tfhe.tfhe_keyswitch_batch(ek, ext[:2], out=ext.view(-1)[(p["N"] + 1):].narrow(0, 0, 2 * row))
    assert ei.value.rc == tfhe.TFHE_EINVAL


def test_buffers_for_a_side_stream_are_allocated_on_it(torch):
    """An output and workspace that the binding allocates for a call on a
    caller-given stream come from that stream's pool: a block just freed on
    the default stream, whose queued kernel will still write it, is not
    handed to the side-stream call (which would see the write land in its
    output)."""
    p = wl.CONFIGS["toy"]["params"]
    sk, ek, ok = keys_for("toy")
    B = 8
    rng = np.random.default_rng(95)
    a, b = rng.integers(0, 2, B), rng.integers(0, 2, B)
    ca = tfhe.to_device(tfhe.tfhe_encrypt_torus(sk, 96, tfhe.encode_bits(a), 0))
    cb = tfhe.to_device(tfhe.tfhe_encrypt_torus(sk, 96, tfhe.encode_bits(b), B))
    ref = tfhe.to_host(tfhe.tfhe_gate_bootstrap_batch(ek, "NAND", ca, cb))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    torch.cuda.synchronize()
    # a default-stream kernel queued behind a bounded spin writes a buffer of
    # the output's size; the buffer is dropped at once, while the write is
    # still queued
    if not hasattr(torch.cuda, "_sleep"):
        pytest.skip("torch has no bounded spin kernel to keep the default stream busy")
    victim = torch.empty((B, p["n"] + 1), dtype=torch.int32, device="cuda:0")
    vptr = victim.data_ptr()
    torch.cuda._sleep(50_000_000)  # a bounded spin on the default stream (20 ms at 2.4 GHz)
    victim.fill_(0x5A5A5A5A)
    del victim
    say("side-stream call while a default-stream write to a freed block is queued")
    out = tfhe.tfhe_gate_bootstrap_batch(ek, "NAND", ca, cb, stream=side)
    same_block = out.data_ptr() == vptr
    torch.cuda.synchronize()
    assert not same_block
    assert np.array_equal(tfhe.to_host(out), ref)
