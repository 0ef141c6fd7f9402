// Checks that programs kept together as one kernel argument stay the
// programs they were: random programs with every kind of pool reference, the
// instructions and the pool words that each refers to equal, and refused
// exactly where instructions, slot tables or pool words do not fit.  Exit
// code 1 on a difference.
#include <stdio.h>
#include <string.h>

#include <random>
#include <vector>

#include "esc.h"
#include "esc_host.h"

using namespace esc;

static std::mt19937 rng(4711);
static int pick(int lo, int hi) { return (int)(lo + rng() % (unsigned)(hi - lo + 1)); }

static Program random_program(int ninsn, int ntables, int nlist)
{
    Program P{};
    P.ninsn = ninsn;
    P.ntables = ntables;
    P.nk = ntables * kSlotTable + nlist;
    for (int i = 0; i < P.nk; i++) P.kpool[i] = (uint32_t)rng();
    for (int i = 0; i < ninsn; i++) {
        Insn &t = P.insn[i];
        t.src = (uint8_t)pick(0, kMaxSlots - 1);
        t.flags = (uint8_t)pick(0, 15);
        t.a = (int32_t)rng(); t.b = (int32_t)rng(); t.c = (int32_t)rng();
        const int kind = pick(0, 3);
        if (kind == 0 && ntables) {
            t.op = pick(0, 1) ? T_IN_HASH : T_IN_BITMAP;
            t.c = pick(0, ntables - 1);
            t.a = t.c * kSlotTable;
        } else if (kind == 1 && nlist) {
            t.op = pick(0, 1) ? T_IN_I32 : T_IN_F32;
            const int at = pick(0, nlist - 1);
            t.a = ntables * kSlotTable + at;
            t.b = pick(0, nlist - at);
        } else {
            const Op ops[] = {T_RANGE_I32, T_RANGE_F32, T_BITSET, U_LOAD, U_ADD, U_MOD, U_SHR};
            t.op = ops[pick(0, 6)];
        }
    }
    return P;
}

static bool same(const Program &P, const ConjPack &k, int part)
{
    if (k.first[part + 1] - k.first[part] != P.ninsn) return false;
    for (int i = 0; i < P.ninsn; i++) {
        const Insn &a = P.insn[i], &b = k.insn[k.first[part] + i];
        if (a.op != b.op || a.src != b.src || a.flags != b.flags || a.b != b.b) return false;
        if (a.op == T_IN_HASH || a.op == T_IN_BITMAP) {
            if (b.c < 0 || b.c >= k.ntables || b.a != b.c * kSlotTable) return false;
            if (memcmp(P.kpool + a.a, k.kpool + b.a, kSlotTable * 4)) return false;
        } else if (a.op == T_IN_I32 || a.op == T_IN_F32) {
            if (a.c != b.c || b.a < k.ntables * kSlotTable || b.a + b.b > kMaxKpool) return false;
            if (memcmp(P.kpool + a.a, k.kpool + b.a, (size_t)a.b * 4)) return false;
        } else if (a.a != b.a || a.c != b.c) {
            return false;
        }
    }
    return true;
}

int main()
{
    int packed = 0, refused = 0;
    for (int it = 0; it < 20000; it++) {
        const int m = pick(1, it % 4 ? 5 : ESC_MAX_CONJ);
        std::vector<Program> progs;
        int ninsn = 0, ntables = 0, nk = 0;
        for (int i = 0; i < m; i++) {
            const int nt = pick(0, 3) ? 0 : pick(0, it % 8 ? 2 : kMaxTables);
            const int room = kMaxKpool - nt * kSlotTable;
            progs.push_back(random_program(pick(0, m > 5 ? 3 : 16), nt, pick(0, 2) ? 0 : pick(0, it % 3 ? room / 4 : room)));
            ninsn += progs.back().ninsn; ntables += progs.back().ntables; nk += progs.back().nk;
        }
        ConjPack k;
        memset(&k, 0xee, sizeof k);
        const bool ok = pack_conjuncts(progs, k);
        if (ok != (ninsn <= kMaxInsns && ntables <= kMaxTables && nk <= kMaxKpool)) {
            printf("fit of %d insns, %d tables, %d words\n", ninsn, ntables, nk);
            return 1;
        }
        if (!ok) { refused++; continue; }
        packed++;
        bool eq = k.ntables == ntables && k.first[0] == 0;
        for (int i = 0; i < m; i++) eq = eq && same(progs[i], k, i);
        if (!eq) { printf("programs differ at iteration %d\n", it); return 1; }
    }
    printf("ok %d packed, %d refused\n", packed, refused);
    return packed > 1000 && refused > 1000 ? 0 : 1;
}
