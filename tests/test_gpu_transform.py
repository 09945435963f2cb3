"""The complex float64 transform of the blind rotation: every form returns the exact integers, also for keys whose
words sit at the ends of their range in patterns that pile up in single transform slots. Tolerance: zero bits (the
rounding error is proven to stay below one half)."""
import numpy as np
import pytest

import oracle
import workloads as W
from paper_2010_09410_amd import client
from paper_2010_09410_amd.device import Context, to_host

pytestmark = pytest.mark.gpu
N = 1024


def extreme_key(pattern):
    """A bootstrapping key [630][6][2][N] (no encryption of anything) of extreme words."""
    g = W.rng(77)
    j = np.arange(N)
    if pattern == "constant":           # the limb split's largest magnitudes, one sign
        row = np.full(N, 0x80000000, np.uint32)
    elif pattern == "alternating":
        row = np.where(j % 2 == 0, 0x80000000, 0x7FFFFFF7).astype(np.uint32)
    elif pattern == "wave":             # square wave of the slowest transform frequency
        row = np.where(np.cos(np.pi * (j + 0.5) / N) >= 0, 0x7FFFFFFF, 0x80000008).astype(np.uint32)
    else:                               # both ends at random
        return g.choice(np.array([0x7FFFFFFF, 0x80000000, 0x7FFFFFF8, 0x80000007], np.uint32), size=(630, 6, 2, N))
    return np.broadcast_to(row, (630, 6, 2, N)).copy()


@pytest.mark.parametrize("pattern", ["constant", "alternating", "wave", "random"])
def test_extreme_keys_equal_oracle_in_every_form(keys, pattern):
    bk = extreme_key(pattern)
    g = W.rng(78)
    B = 3
    ops = np.array([W.NAND, W.XOR, W.ORNOT], np.uint8)
    enc = W.tlwe_draws(g, 2 * B)
    x = client.tlwe_encrypt_bits(keys["s0"], g.integers(0, 2, 2 * B), *enc)
    ref = oracle.gates(bk, keys["ksk"], ops, x[:B], x[B:])
    with Context(bk, keys["ksk"]) as ctx:
        d = ctx.tensor(ops), ctx.tensor(x[:B]), ctx.tensor(x[B:])
        for form in (3, 4, 8):
            ctx.set_tuning(B, form, 2)
            np.testing.assert_array_equal(to_host(ctx.gates(*d)), ref, err_msg=f"{pattern}, form {form}")
        out, _ = ctx.gates_key_copies(*d, waves=8, copies=2)    # per-gate keys
        np.testing.assert_array_equal(to_host(out), ref, err_msg=f"{pattern}, key copies")
        ctx.sync()


@pytest.mark.parametrize("B", [1, 3, 4, 5, 8, 9, 13])
def test_shared_key_workgroups_with_idle_waves(gpu, keys, B):
    """Batches that leave waves of a workgroup without a gate, and gates that do not bootstrap, in the forms whose
    workgroups stream the key together."""
    g = W.rng(79 + B)
    ops = g.choice(np.array([W.NAND, W.NOT, W.XNOR, W.AND], np.uint8), size=B)
    x = client.tlwe_encrypt_bits(keys["s0"], g.integers(0, 2, 2 * B), *W.tlwe_draws(g, 2 * B))
    d = gpu.tensor(ops), gpu.tensor(x[:B]), gpu.tensor(x[B:])
    _, ks = gpu.tuning(B)
    outs = []
    try:
        for form in (33, 3, 4, 8):
            gpu.set_tuning(B, form, ks)
            outs.append(to_host(gpu.gates(*d)))
    finally:
        gpu.set_tuning(B, 0, ks)
    for o in outs[1:]:
        np.testing.assert_array_equal(o, outs[0])


# operand words whose three gadget digits are all -32 or all 31
LOW, HIGH = np.uint32(0x7DF7E000), np.uint32(0x7DF7A000)


def test_extreme_external_products_equal_oracle(gpu):
    """Digits and key words at the ends of their ranges, in the sign patterns (constant, alternating, a slow square wave,
    random) whose products pile up in single coefficients or single transform slots."""
    g = W.rng(81)
    j = np.arange(N)
    signs = [np.ones(N, bool), j % 2 == 0, np.cos(np.pi * (j + 0.5) / N) >= 0, g.integers(0, 2, N) == 1]
    C, x = [], []
    for a in signs:
        for b in signs:
            key = np.where(a, np.uint32(0x7FFFFFF7), np.uint32(0x80000000))
            C.append(np.broadcast_to(key, (6, 2, N)))
            x.append(np.broadcast_to(np.where(b, HIGH, LOW), (2, N)))
    C, x = np.ascontiguousarray(C), np.ascontiguousarray(x)
    out = to_host(gpu.debug_external_product(gpu.tensor(C), gpu.tensor(x)))
    for i in range(len(C)):
        np.testing.assert_array_equal(out[i], oracle.external_product(C[i], x[i]), err_msg=f"pair {i}")


def random_words(gpu, seed, *shape):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randint(-(1 << 31), 1 << 31, shape, generator=gen, device="cuda", dtype=torch.int32)


def test_ram_reads_in_chunks_and_shared_selectors(gpu):
    """Reads beyond one launch sequence (2^14 / v of them) and tree levels whose CMUX count per read is no multiple of
    eight give what each read gives by itself (one wave per CMUX, pinned by the oracle in test_gpu_memory.py)."""
    ram, addr = random_words(gpu, 1, 1, 4, 2, N), random_words(gpu, 2, 8200, 2, 6, 2, N)
    out = to_host(gpu.ram_read(ram, addr))
    for r in (0, 8191, 8192, 8199):
        np.testing.assert_array_equal(out[r], to_host(gpu.ram_read(ram, addr[r:r + 1]))[0], err_msg=f"read {r}")
    ram, addr = random_words(gpu, 3, 5, 8, 2, N), random_words(gpu, 4, 300, 3, 6, 2, N)   # 20, 10, 5 CMUXes per read
    out = to_host(gpu.ram_read(ram, addr))
    for r in (0, 7, 299):
        np.testing.assert_array_equal(out[r], to_host(gpu.ram_read(ram, addr[r:r + 1]))[0], err_msg=f"read {r}")


def test_extreme_level2_key_equals_oracle(gpu, keys):
    """Circuit bootstrapping with a level-2 key whose three limbs all sit at the ends of their ranges, constant, alternating,
    as a slow square wave and at random by row; the private key-switching key is random words."""
    g = W.rng(82)
    j = np.arange(2048)
    limbs = lambda l0, l1, l2: np.uint64((l0 + (l1 << 22) + (l2 << 44)) % (1 << 64))  # noqa: E731
    low, high = limbs(-(1 << 21), -(1 << 21), -(1 << 19)), limbs((1 << 21) - 1, (1 << 21) - 1, (1 << 19) - 1)
    signs = [np.ones(2048, bool), j % 2 == 0, np.cos(np.pi * (j + 0.5) / 2048) >= 0, g.integers(0, 2, 2048) == 1]
    rows = np.stack([np.stack([np.where(signs[(r + o) % 4], high, low) for o in range(2)]) for r in range(8)])
    bk2 = np.ascontiguousarray(np.broadcast_to(rows, (630, 8, 2, 2048)))
    pksk = g.integers(0, 2 ** 32, size=(2, 2049, 12, 3, 2, N), dtype=np.uint32)
    c = client.tlwe_encrypt_bits(keys["s0"], np.array([1]), *W.tlwe_draws(g, 1))
    want = oracle.circuit_bootstraps(bk2, pksk, c)
    key = gpu.cbkey(bk2, pksk)
    try:
        np.testing.assert_array_equal(to_host(key.bootstrap(gpu.tensor(c)))[0].reshape(6, 2, N), want[0])
    finally:
        key.close()


def test_private_key_switch_batches_equal_single_inputs(gpu, keys):
    """Batch sizes on both sides of every tile width of the private key switch (three rows of it per input; 16, 32, 64 and 128
    rows) and past one launch of it (8,192 rows): each input's output is what it gives alone, a batch of one the oracle's."""
    g = W.rng(83)
    bk2 = g.integers(0, 2 ** 64, size=(630, 8, 2, 2048), dtype=np.uint64)
    pksk = g.integers(0, 2 ** 32, size=(2, 2049, 12, 3, 2, N), dtype=np.uint32)
    c = g.integers(0, 2 ** 32, size=(2740, 631), dtype=np.uint32)
    want = oracle.circuit_bootstraps(bk2, pksk, c[:1])
    key = gpu.cbkey(bk2, pksk)
    try:
        d = gpu.tensor(c)
        alone = {r: to_host(key.bootstrap(d[r:r + 1]))[0] for r in (0, 4, 5, 9, 10, 20, 21, 41, 42, 2729, 2730, 2731, 2739)}
        np.testing.assert_array_equal(alone[0].reshape(6, 2, N), want[0])
        for R in (5, 6, 10, 11, 21, 22, 42, 43, 2740):
            out = to_host(key.bootstrap(d[:R]))
            for r in (x for x in alone if x < R):
                np.testing.assert_array_equal(out[r], alone[r], err_msg=f"input {r} of {R}")
    finally:
        key.close()


@pytest.mark.parametrize("B", [1, 16, 17, 96, 97, 192, 193, 384, 385, 768, 769, 1030, 2433])
def test_matrix_core_key_switch_equals_the_gathering_one(gpu, B):
    """Both sides of every tile width of the matrix-core key switch and of a last tile, against the form that gathers the
    key rows of each gate; a third of the gates does not bootstrap and keeps its row."""
    g = W.rng(84 + B)
    ops = g.choice(np.array([W.NAND, W.NOT, W.XNOR], np.uint8), size=B)
    ops[-1] = W.NAND
    d = gpu.tensor(ops), random_words(gpu, B, B, 631), random_words(gpu, B + 1, B, 631)
    _, ks = gpu.tuning(B)
    outs = []
    try:
        for form in (0, 3):
            gpu.set_tuning(B, 0, form)
            outs.append(to_host(gpu.gates(*d)))
    finally:
        gpu.set_tuning(B, 0, ks)
    np.testing.assert_array_equal(outs[1], outs[0])


def test_chains_on_a_workgroup_equal_those_on_a_wave(gpu):
    """Up to two CMUX chains per compute unit (512 here) take a workgroup each: reads and write bars just above the line,
    one wave each, give what the same ones give below it (pinned by the oracle in test_gpu_memory.py)."""
    v, w = 7, 64                                        # two cells a ROM polynomial pair, rotations of 64 << j
    rom, addr = random_words(gpu, 5, 8, 2, N), random_words(gpu, 6, 513, v, 6, 2, N)
    out = to_host(gpu.rom_read(rom, addr, v, w))
    for a, b in ((0, 512), (1, 513), (511, 512)):       # tree levels of 4, 2 and 1 per read, rotations
        np.testing.assert_array_equal(out[a:b], to_host(gpu.rom_read(rom, addr[a:b].contiguous(), v, w)))
    ram, sel = random_words(gpu, 7, 3, 256, 2, N), random_words(gpu, 8, 8, 6, 2, N)       # 768 bars against 512
    flag, data = random_words(gpu, 9, 631), random_words(gpu, 10, 3, 631)
    whole, part = ram.clone(), ram[:2].contiguous().clone()
    gpu.ram_write(whole, sel, flag, data)
    gpu.ram_write(part, sel, flag, data[:2].contiguous())
    np.testing.assert_array_equal(to_host(whole)[:2], to_host(part))


@pytest.mark.parametrize("B", [511, 512, 513, 769, 1023])
def test_pairs_of_gates_equal_single_ones(gpu, B):
    """Workgroups of two gates (whole rounds of two per compute unit, an odd last pair) and the mixture with workgroups of
    one gate give what the key-sharing form gives; a third of the gates does not bootstrap."""
    g = W.rng(85 + B)
    ops = g.choice(np.array([W.NAND, W.NOT, W.XNOR], np.uint8), size=B)
    d = gpu.tensor(ops), random_words(gpu, B + 2, B, 631), random_words(gpu, B + 3, B, 631)
    _, ks = gpu.tuning(B)
    outs = []
    try:
        for form in (8, 4, 3):
            gpu.set_tuning(B, form, ks)
            outs.append(to_host(gpu.gates(*d)))
    finally:
        gpu.set_tuning(B, 0, ks)
    for o in outs[1:]:
        np.testing.assert_array_equal(o, outs[0])


def test_a_tuning_measured_with_other_kernels_is_measured_again(gpu, tmp_path):
    """A cache entry without the mark of these kernels, or with another one, is ignored and rewritten."""
    import json
    buckets = (1, 16, 64, 256, 1024, 2048, 4096)
    saved = {b: gpu.tuning(b)[1] for b in buckets}
    path = tmp_path / "tune.json"
    try:
        gpu.autotune(max_batch=64, cache_path=str(path))
        (key, entry), = json.loads(path.read_text()).items()
        mark = entry.pop("kernels")
        for other in ({}, {"kernels": [mark[0] - 1]}):
            path.write_text(json.dumps({key: {**entry, **other, "br_round_ms": [99.0] * 5}}))
            gpu.autotune(max_batch=64, cache_path=str(path))
            again = json.loads(path.read_text())[key]
            assert again["kernels"] == mark and again["br_round_ms"] != [99.0] * 5
    finally:
        for b, t in saved.items():
            gpu.set_tuning(b, 0, t)


def test_external_products_past_one_chunk(gpu):
    """More external products than are transformed at once (2^14): each is what it is alone."""
    J = (1 << 14) + 3
    C, x = random_words(gpu, 11, J, 6, 2, N), random_words(gpu, 12, J, 2, N)
    out = to_host(gpu.debug_external_product(C, x))
    for j in (0, (1 << 14) - 1, 1 << 14, J - 1):
        np.testing.assert_array_equal(out[j], to_host(gpu.debug_external_product(C[j:j + 1].contiguous(), x[j:j + 1].contiguous()))[0])


def test_workgroups_without_a_bootstrap_end_at_once(gpu):
    """Workgroups of the key-sharing form none of whose gates bootstraps: no pass over the key for 2,048 NOT gates through
    the allocation-free entry point (0.3 ms with launches, where a round of the blind rotation takes 12), and among others
    the words of the form with a gate per workgroup."""
    import torch
    from paper_2010_09410_amd import _native as nv
    B = 2048
    a, b = random_words(gpu, 13, B, 631), random_words(gpu, 14, B, 631)
    out = torch.empty_like(a)
    times = {}
    for op in (W.NOT, W.NAND):
        ops = torch.full((B,), int(op), dtype=torch.uint8, device="cuda")
        for _ in range(3):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record()
            nv.vsp_gates_noalloc(gpu.handle, ops.data_ptr(), a.data_ptr(), b.data_ptr(), out.data_ptr(), B, nv.VSP_BATCHED,
                                 gpu.stream())
            t1.record()
            t1.synchronize()
            times[op] = min(times.get(op, 1e9), t0.elapsed_time(t1))
        if op == W.NOT:
            np.testing.assert_array_equal(to_host(out), (0 - to_host(a).astype(np.int64)).astype(np.uint32))
    assert times[W.NOT] < times[W.NAND] / 8, times
    ops = np.full(61, W.NAND, np.uint8)
    for lo, hi in ((0, 8), (10, 32), (40, 48), (56, 61)):      # whole workgroups of eight, parts of others, the ragged last
        ops[lo:hi] = W.NOT
    d = gpu.tensor(ops), a[:61].contiguous(), b[:61].contiguous()
    _, ks = gpu.tuning(61)
    outs = []
    try:
        for form in (3, 8):
            gpu.set_tuning(61, form, ks)
            outs.append(to_host(gpu.gates(*d)))
    finally:
        gpu.set_tuning(61, 0, ks)
    np.testing.assert_array_equal(outs[1], outs[0])


@pytest.mark.parametrize("pattern", ["constant", "alternating", "wave", "random"])
def test_extreme_keys_in_workgroups_of_two_gates(keys, pattern):
    """One gate more than compute units in form 4: all of them, an odd last one too, run on workgroups of two gates, whose
    first exchange goes through registers."""
    import torch
    bk = extreme_key(pattern)
    g = W.rng(86)
    ops = np.array([W.NAND, W.XOR, W.ORNOT], np.uint8)
    x = client.tlwe_encrypt_bits(keys["s0"], g.integers(0, 2, 6), *W.tlwe_draws(g, 6))
    ref = oracle.gates(bk, keys["ksk"], ops, x[:3], x[3:])
    B = torch.cuda.get_device_properties(0).multi_processor_count + 1
    of = np.arange(B) % 3
    with Context(bk, keys["ksk"]) as ctx:
        ctx.set_tuning(B, 4, 3)
        out = to_host(ctx.gates(ctx.tensor(ops[of]), ctx.tensor(x[of]), ctx.tensor(x[3 + of])))
        ctx.sync()
    np.testing.assert_array_equal(out, ref[of])


def test_extreme_words_in_every_shape_of_the_cmux_memory(gpu, keys):
    """Selectors and cell differences at the ends of their ranges through CMUXes that share a selector, on a workgroup and
    on a wave each, and through ROM rotations in workgroups of eight waves (2,049 reads), of one, and on a workgroup."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    g = W.rng(87)
    j = np.arange(N)
    signs = [np.ones(N, bool), j % 2 == 0, np.cos(np.pi * (j + 0.5) / N) >= 0, g.integers(0, 2, N) == 1]
    sel = np.stack([np.broadcast_to(np.where(s, np.uint32(0x7FFFFFF7), np.uint32(0x80000000)), (6, 2, N)) for s in signs])
    word = np.stack([np.broadcast_to(np.where(s, HIGH, LOW), (2, N)) for s in signs])
    ram = np.zeros((8, 2, 2, N), np.uint32)             # bits 0-3: cells 0 and x, bits 4-7: -x and 0
    ram[:4, 1], ram[4:, 0] = word, (1 << 32) - word.astype(np.uint64)
    addr = gpu.tensor(np.ascontiguousarray(sel[np.arange(cus + 1) % 4, None]))
    ref = oracle.ram_reads(keys["ksk"], ram, sel[:, None])
    for R in (cus + 1, cus // 2, 4):                    # 8 CMUXes a read
        out = to_host(gpu.ram_read(gpu.tensor(ram), addr[:R].contiguous()))
        np.testing.assert_array_equal(out, ref[np.arange(R) % 4], err_msg=f"{R} RAM reads")
    v, w = 5, 32                                        # blocks of 32 that change sign: X^-32 P - P = -2 P = LOW, -LOW
    half = np.uint32(((1 << 32) - int(LOW)) // 2)
    rom = np.broadcast_to(np.where((j // 32) % 2 == 0, half, (0 - half.astype(np.int64)).astype(np.uint32)), (1, 2, N))
    rom = np.ascontiguousarray(rom)
    R = 8 * cus + 1
    sels = np.ascontiguousarray(np.broadcast_to(sel[:, None], (4, v, 6, 2, N)))
    addr = gpu.tensor(sels)[torch.arange(R, device="cuda") % 4].contiguous()
    ref = oracle.rom_reads(keys["ksk"], rom, sels)
    for n in (R, 2 * cus + 1, 4):
        out = to_host(gpu.rom_read(gpu.tensor(rom), addr[:n].contiguous(), v, w))
        np.testing.assert_array_equal(out, ref[np.arange(n) % 4], err_msg=f"{n} ROM reads")


def test_shared_selectors_in_several_rounds(gpu):
    """Tree levels whose workgroups take several groups of eight CMUXes in turn, with a remainder: 52 per read in four rounds
    of two workgroups, then 26 in two rounds (on 256 compute units), against reads alone, whose CMUXes take a workgroup each."""
    import torch
    R = torch.cuda.get_device_properties(0).multi_processor_count // 2
    ram, addr = random_words(gpu, 15, 13, 8, 2, N), random_words(gpu, 16, R, 3, 6, 2, N)
    out = to_host(gpu.ram_read(ram, addr))
    for r in (0, 1, R // 2, R - 1):
        np.testing.assert_array_equal(out[r], to_host(gpu.ram_read(ram, addr[r:r + 1].contiguous()))[0], err_msg=f"read {r}")
