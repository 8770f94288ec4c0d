"""Which work may run at the same time when analyses of one context go to several streams: the scratch that
sali_workspace_bytes asks for and the waits between batches, against each other, on the CPU."""
import pytest

LANES = 32                                       # SALI_ANALYSIS_LANES


def _expansion_slots(tiles):
    """Slots of the ring of expansions: nothing else of the scratch depends on the tiles per frame."""
    from paper_2602_14236_amd import binding
    h = w = 96                                   # one level: 96 x 96 float4 + float, both a multiple of 256 bytes
    size = {t: binding.workspace_bytes(binding.make_config(h, w, flow_levels=1, tiles_per_frame=t))[0] for t in (1, tiles)}
    more, rest = divmod(size[tiles] - size[1], h * w * 20)
    assert rest == 0
    return LANES + 1 + more


@pytest.mark.parametrize("tiles,entries", [(1, 1), (1, 16), (2, 2), (2, 16), (3, 3), (3, 15), (4, 16), (8, 8), (8, 16)])
@pytest.mark.parametrize("streams", [2, 3])
def test_no_expansion_is_overwritten_before_its_last_reader(tiles, entries, streams):
    """Batches of `entries` analyses in turn on `streams` streams.  A batch is three pieces of work on its stream: its
    expansions (after the analysis LANES before its last is done), its flow (after the expansions of the batch before),
    its tiers (after those of the batch before).  Entry n's expansion lies in slot n % slots and is read by the flows of
    n and of n + tiles; whoever writes the slot next must be ordered behind both."""
    slots = _expansion_slots(tiles)
    batches = 8 * LANES // entries + 3
    before = {}                                  # piece -> all that is ordered before it
    tail_of_stream = {}

    def add(piece, stream, *waits):
        before[piece] = set()
        for p in (tail_of_stream.get(stream),) + waits:
            if p is not None:
                before[piece] |= before[p] | {p}
        tail_of_stream[stream] = piece

    for b in range(batches):
        last = (b + 1) * entries - 1
        old = (("tiers", (last - LANES) // entries),) if last >= LANES else ()
        prev = (lambda piece: ((piece, b - 1),) if b else ())
        add(("expand", b), b % streams, *old)
        add(("flow", b), b % streams, *prev("expand"))
        add(("tiers", b), b % streams, *prev("tiers"))
    for n in range(batches * entries - slots):
        write = ("expand", (n + slots) // entries)
        for reader in (n, n + tiles):
            assert ("flow", reader // entries) in before[write], \
                f"entry {n + slots} may overwrite slot {n % slots} while the flow of entry {reader} reads it"
