// The two ways in which the device's words come to the host, in one mailbox (host code only; nothing here runs on a GPU).  Prints one line
// per check that failed, then "checked <n>".
#include <cstdio>
#include "../paper_2306_16354_amd/csrc/slhc_api.hip"

int main()
{
    alignas(64) static unsigned char memory[Mailbox::BYTES];
    long checked = 0;
    auto expect = [&](bool got, bool want, const char* what, unsigned seq) {
        if (got != want) std::printf("%s, message %u: %s\n", what, seq, got ? "taken for arrived" : "not seen");
        ++checked;
    };
    Mailbox m(nullptr);
    m.box.p = memory;
    const int n = slhc::CSR_TOLD;
    for (int turn = 0; turn < 100; ++turn) {
        // a round's words, each one the number of the message that follows
        const uint32_t round = m.next();
        for (int i = 0; i < n; ++i) {
            expect(m.arrived_tagged(n), false, "round", round);
            m.tagged()[i] = ((unsigned long long)round << 32) | (round + 1);
        }
        expect(m.arrived_tagged(n), true, "round", round);
        // a fetch behind it, of words that are the number of the next round
        const uint32_t fetch = m.next();
        expect(m.arrived(), false, "fetch", fetch);
        for (int i = 0; i < Mailbox::WORDS; ++i) m.words()[1 + i] = fetch + 1;
        expect(m.arrived(), false, "fetch", fetch);
        m.words()[0] = fetch;
        expect(m.arrived(), true, "fetch", fetch);
    }
    if (m.words() + 1 + Mailbox::WORDS > reinterpret_cast<uint32_t*>(memory + sizeof(memory))) std::printf("words beyond the box\n");
    m.box.p = nullptr;
    std::printf("checked %ld\n", checked);
    return 0;
}
